// How launches are planned: plain host functions of the call's sizes, so that they can be checked without a GPU.
#pragma once

#include <algorithm>

namespace mp {

// Upper bound of the keys a decode call selects per unit: the selected clusters fit the key budget, and with two levels
// they are children of the promising clusters, which fit the coarse budget.  (The launch is cut by this bound: by the key
// budget alone, a coarse budget of an eighth of it left seven of eight workgroups without rows -- 128 units, budgets
// 32768 / 4096, 4 heads, whole step 153 us, now 66; 64 units 95, now 43.)
inline int most_selected(int levels, int key_budget, int coarse_budget, int n_tokens)
{
    const int most = std::min(key_budget, n_tokens);
    return levels == 2 ? std::min(most, coarse_budget) : most;
}

// Matrix-core kernel: workgroups per unit for a launch over all units.  One workgroup per compute unit: four waves
// with three pieces of 4 KiB each on their way keep a compute unit's share of the memory system busy, and every
// further workgroup only adds a prologue, an epilogue and partials to merge.  Measured (dense, us by workgroups in
// all): 64 units x 60013 rows, 8 heads: 128: 348, 256: 292, 512: 295, 1024: 306, 4032: 330; 8 x 32768, 4 heads:
// 128: 29.9, 256: 25.8, 512: 27.8, 1024: 37.8; 1 x 131072: 128: 21.0, 256: 20.4, 512: 26.8; selected keys, whole
// step: 128 units x 8192: 128: 152, 256: 125, 512: 123.5, 1024: 125.8; 24 x 6250, 8 heads: 120: 56.3, 240: 49.4,
// 480: 51.0, 792: 57.2.
//
// Two thirds of the compute units are enough (170 workgroups reach what 256 do), a few more workgroups than compute units
// are not (some then have two, and these are the call's time).  So: as many per unit as fit one round, unless two rounds
// (both resident at once) leave no more than three quarters of its rows to the busiest compute unit: 129 to 170 units,
// and others where a long tail makes the shares uneven.  Dense, 32768 rows, 4 heads, us by
// workgroups per unit: 86 units 2: 222, 3: 305, 5: 214; 96: 2: 243, 3: 314, 4: 252; 129: 1: 389, 2: 461, 3: 330; 144: 1:
// 398, 2: 465, 3: 353; 160: 1: 415, 2: 486, 3: 392; 176: 1: 438, 2: 508; 192: 1: 476, 2: 509.
// More units than compute units: the count (of up to six rounds) whose last round is fullest; 264 units 1: 883, 2: 756,
// 3: 714, 5: 707; 320: 2: 793, 3: 778, 4: 816.
constexpr int kStreamWgs = 256;
inline int fullest_rounds(int n_units)
{
    int best = 1;
    double best_fill = 0.0;
    for (int c = 1; c == 1 || (long long)c * n_units <= 6 * kStreamWgs; ++c) {
        const long long wgs = (long long)c * n_units, rounds = (wgs + kStreamWgs - 1) / kStreamWgs;
        const double fill = (double)wgs / (double)(rounds * kStreamWgs);
        if (fill > best_fill + 0.03) {      // (fewer workgroups where it is much the same)
            best = c;
            best_fill = fill;
        }
    }
    return best;
}

// Most chunks a unit's rows are cut into (a short stream's chunk on top: one more).
inline int most_stream_chunks(int n_units)
{
    return n_units <= kStreamWgs ? 2 * kStreamWgs / n_units : fullest_rounds(n_units);
}

// Rows per chunk when n rows are cut into at most `chunks` chunks of about the same size: a multiple of 64 (16 rows a wave
// and tile).
inline int stream_chunk_rows(long long n, int chunks)
{
    const long long per = (n + chunks - 1) / chunks;
    return (int)std::max<long long>(64, (per + 63) / 64 * 64);
}

// Rows of the longest chunk when two streams are cut into `chunks` chunks together.  A stream of up to half a chunk is one
// chunk on top of them and takes none away from the other.
inline int longest_chunk(long long first, long long tail, int chunks)
{
    const int of_first = stream_chunk_rows(first, chunks), of_tail = stream_chunk_rows(tail, chunks);
    if (2 * tail <= of_first) return of_first;
    if (2 * first <= of_tail) return of_tail;
    if (chunks == 1) return std::max(of_first, of_tail);
    const int share = (int)(chunks * first / (first + tail));
    int best = 0;
    for (int k = std::max(1, share); k <= std::max(1, share) + 1 && k < chunks; ++k) {
        const int rows = std::max(stream_chunk_rows(first, k), stream_chunk_rows(tail, chunks - k));
        if (best == 0 || rows < best) best = rows;
    }
    return best ? best : std::max(stream_chunk_rows(first, chunks - 1), stream_chunk_rows(tail, 1));
}

// Rows per chunk of the selected keys (or centroid terms, or a dense call's keys) and of the tail; `most` limits the chunks
// of each.  (A short tail took one of two chunks from units 86 to 128: 96 units, 2048 keys, tail of 130, 4 heads, whole
// step 57 us, now 42.  A third chunk of the same length for it is as bad where it is long: 96 units, 512 keys, tail of 1500,
// 1 head 43.4 -> 38 us.)  Each stream's chunks are cut evenly, so that a short one's rows are spread over its four waves.
struct StreamPlan {
    int first_rows, tail_rows;
};
inline StreamPlan plan_streams(int n_units, long long first, long long tail, int most = 1 << 20)
{
    int rows = 0;
    if (n_units > kStreamWgs) {
        rows = longest_chunk(first, tail, std::min(most, fullest_rounds(n_units)));
    } else {
        long long best = 0;      // rows of the busiest compute unit
        for (int r = 1; r <= 2; ++r) {
            const int t = longest_chunk(first, tail, std::min(most, r * kStreamWgs / n_units));
            // (a stream of up to half a chunk does not count)
            const long long chunks = (2 * first > t ? (first + t - 1) / t : 0) + (2 * tail > t ? (tail + t - 1) / t : 0);
            const long long busiest = (chunks * n_units + kStreamWgs - 1) / kStreamWgs * t;
            if (r == 1 || 4 * busiest <= 3 * best) {
                rows = t;
                best = busiest;
            }
        }
    }
    auto even = [&](long long n) { return stream_chunk_rows(n, (int)std::max<long long>(1, (n + rows - 1) / rows)); };
    return StreamPlan{even(first), even(tail)};
}

// Centroid terms that a decode step leaves to the value pass per unit, about (as if all clusters were of one size).
inline long long likely_terms(int levels, int n_tokens, int n_fine, int n_coarse, int key_budget, int coarse_budget)
{
    const long long n = std::max(n_tokens, 1), candidates = levels == 2 ? std::min<long long>(coarse_budget, n) : n;
    const long long taken = std::min<long long>(key_budget, candidates);
    return (n_fine * (candidates - taken) + (levels == 2 ? n_coarse * (n - candidates) : 0)) / n;
}

// Whether the terms that ride along with the selected keys have a wave of their own (bf16 rows): where every workgroup has a compute
// unit (its ten waves do not share one with ten others: 130 units, two workgroups each, 47.1 -> 47.4 to 48.8 us, 300 units 62.5 ->
// 68.5; a tail of up to half a chunk, one workgroup a unit on top, can be what is too many: 24 units of 6250 keys and a tail of 201 have
// 264); and where that wave has no more rows than the others, or than one fetch of row numbers brings, as far as one can tell.
// Whole step, us, riding / own wave: 1 unit of 4 heads x 512 keys 21.0 / 19.4; 8 x 4096 24.5 / 23.5; 32 x 4096 of 5 heads 37.6 / 36.5; 32 x
// 2048 and a tail of 200 35.7 / 34.1; 100 x 2048 39.0 / 37.7; 128 x 8192 (256 terms a workgroup, 1024 keys a wave) 120.3 / 118.5.
// The line, one level, terms a workgroup by keys a wave, clusters of one size: 1 x 1024 (28 by 16) 25.15 / 24.13; 8 x 2048 (32 by 16)
// 60.9 / 59.6; 8 x 4096 (59 by 32) 69.6 / 69.1; 64 x 4096 (237 by 256) 94.3 / 93.3; 128 x 2048 (250 by 256) 56.5 / 55.4, (300 by 256) 77.7 /
// 77.8; 32 x 4096 (188 by 128) 109.0 / 109.3, of 8 heads 132.3 / 133.0.  Where a few large clusters are selected and hold half of all keys,
// twice as many terms stay behind: 8 x 2048 (64 by 16) 51.5 / 51.6; 8 x 4096 (47 by 32) 46.9 / 46.0; 32 x 4096 (237 by 128) 66.3 / 66.4, (375
// by 128) 94.4 / 96.3; 64 x 4096 (474 by 256) 87.0 / 89.9; 128 x 2048 (398 by 256) 53.4 / 54.7, (498 by 256) 57.6 / 60.7, (598 by 256) 74.1 / 78.5.
inline bool terms_have_a_wave(long long workgroups, long long terms, long long key_chunks, int chunk_rows)
{
    const int most = std::min(chunk_rows / 2, std::max(chunk_rows / 4, 64));
    return workgroups <= kStreamWgs && terms <= key_chunks * most;
}

// Dense calls of one head to a unit over few rows: the vector-ALU kernel, in the same chunks.  Such a call is one chain of
// latencies, and its chain is as short or shorter: no staging in LDS, and the work of an epilogue grows with the heads.  Us on the
// device, here / matrix cores, 1 head: 8 units x 2000 rows 8.7 / 9.0, 8 x 8192 10.7 / 10.9, 32 x 4096 14.2 / 14.4, 64 x 500 9.9 / 10.2, 128 x 500
// 10.8 / 10.9, 64 x 2000 14.6 / 14.4, 128 x 1000 14.75 / 14.3, 1 x 8192 9.2 / 9.1, 1 x 200 6.8 / 6.6; at 131072 rows in all the two have met
// (32 x 8192 28.1 / 26.4 before the matrix cores' kernel had its arguments in registers).  With two heads the matrix cores win everywhere
// since then: 1 x 200 7.9 / 6.9, 1 x 8192 10.6 / 9.4, 8 x 64 6.65 / 5.4, 8 x 2000 10.3 / 9.1, 8 x 8192 11.7 / 11.5, 32 x 4096 16.4 / 15.2, 64 x 500
// 10.7 / 10.3, 64 x 2000 16.5 / 15.0, 128 x 100 7.7 / 6.6, 300 x 400 16.8 / 15.2.
inline bool short_dense_on_vector_alu(int group, int n_units, long long n)
{
    return group == 1 && n_units * n <= 131072;
}

// Selected keys stored as 8-bit rows, one query head to a unit: the vector-ALU kernel.  A row's sixteen columns of the matrix
// product would hold three parts of one head; the conversions are for all sixteen.  Whole step, us, here / matrix cores, 1 head:
// 8 units x 4096 keys 25.3 / 25.4, 32 x 4096 29.6 / 30.5, 64 x 4096 36.4 / 36.6, 128 x 4096 50.1 / 50.3; 2 heads: 8 x 4096 27.2 /
// 26.4, 32 x 4096 32.0 / 31.4, 128 x 8192 77.8 / 74.6; 4 heads: 128 x 4096 64.3 / 52.0; 8 heads: 64 x 4096 67.3 / 42.3.
inline bool bytes_on_vector_alu(int group) { return group == 1; }

// Workgroups per unit that work out the logits of all fine clusters while the unit's own workgroup scores its coarse level (two
// levels; 0: none).  They pay where they are done by the time the candidates are known: at most two rounds of 128 clusters
// each, on compute units that are idle otherwise, and ten megabytes of centroid rows in all (more of them slow the coarse level's
// down).  Whole step, us, without / with, four heads unless said otherwise: 1 unit x 1024 clusters 25.5 / 23.5; 8 x 256 22.9 /
// 22.2, x 1024 27.7 / 25.6 (128 clusters a helper; 25.8 with 256, 28.5 with 512), x 1024 of 8 heads 31.5 / 29.1, x 2048 33.4 /
// 28.0 (34.3 with 512 a helper), x 4096 37.6 / 33.1; 16 x 2048 31.3 / 29.7; 24 x 1562 41.3 / 37.3, of 8 heads 47.0 / 41.3; 32 x 1024 36.0 /
// 34.4; 40 x 937 of 6 heads 41.7 / 40.2; 64 x 320 29.0 / 28.6; no gain: 64 x 640 37.6 / 37.9 (10.5 MB), 32 x 2048 of 5
// heads 39.6 / 41.5 (16.8 MB).
constexpr int kHelpedClusters = 40000;      // of all units together
inline int score_helpers(int n_units, int n_compute_units, int levels, int n_fine)
{
    const int spare = n_units > 0 ? (n_compute_units - n_units) / n_units : 0;
    if (levels != 2 || spare < 1 || (long long)n_units * n_fine > kHelpedClusters) return 0;
    const int most = std::min(spare, (n_fine + 127) / 128);
    return (n_fine + most - 1) / most <= 256 ? most : 0;
}

// Whether they are launched.  A unit takes their logits if its candidates fit the register path (1024), as many as a budget of keys is likely
// to leave (with a sixteenth to spare: a unit has a few less or more).  With more candidates they only bring the rows nearer, which pays up
// to 32768 clusters of all units: without / with, all clusters candidates, 1 unit x 4096 105.0 / 103.0; 8 x 2048 67.4 / 65.7, x 4096 107.7 /
// 105.8; 9 x 2048 69.7 / 68.4, x 4096 109.8 / 118.8, of 2 heads 133.2 / 139; 16 x 2048 71.4 / 69.9; 24 x 1300 63.4 / 62.0, x 1600 of 8
// heads 79.0 / 79.6; 28 x 1300 65.7 / 65.6; 9 x 4096, 1169 candidates 60.5 / 61.2, 877 47.4 / 39.4; 24 x 1600 of 8 heads, 952 49.6 / 39.3.
inline bool helpers_pay(int n_units, int n_tokens, int n_fine, int coarse_budget)
{
    const int n = std::max(n_tokens, 1);
    const long long candidates = (long long)n_fine * std::min(coarse_budget, n) / n;
    return candidates <= 1024 + 64 || (long long)n_units * n_fine <= 32768;
}

// Waves of a workgroup of an assignment step that looks at all centroids, where two workgroups of eight fit a compute unit: sixteen up to
// 256 (block, unit) pairs, unless whole workgroups of them come to less than four fifths of the waves that eight come to.
inline int waves_for_blocks(long long pairs)
{
    if (pairs < 1 || pairs > 256) return 8;
    return 5 * (256 / pairs) > 2 * (512 / pairs) ? 16 : 8;
}

// Whether the coarse level of (block, unit) pairs of at most max_pts fine and max_k coarse clusters runs in one launch, one
// workgroup per pair, or in a launch per step.  The workgroup's time grows with its clusters (each is one wave's walk over
// all points and a trip to memory, sixteen or eight waves) and points, that of the steps with their number and, beyond one
// round of workgroups, the pairs.  Whole build of ten iterations, one launch / steps, us:
//   1 pair     256 points x 32: 552 / 627,   x 64: 576 / 572,   x 256: 864 / 472;   512 x 32: 789 / 818, x 64: 865 / 732
//   64 pairs   160 points x 64: 595 / 612,   x 96: 620 / 603;   256 x 48: 761 / 851, x 64: 804 / 831, x 96: 814 / 795;
//              512 x 48: 1328 / 1408,        x 64: 1437 / 1392, x 256: 1754 / 1295
//   256 pairs  256 points x 96: 1352 / 1437, x 256: 1577 / 1586; 512 x 48: 2499 / 2682, x 128: 2683 / 2658
//   1024 pairs 256 points x 64: 5035 / 5092, x 128: 5462 / 5428; 512 x 48: 8509 / 8640, x 64: 8983 / 8688
// These are from before the points stood in LDS and touched clusters alone were summed again.  With that, one launch is the shorter way at
// five of six points past the lines, too, one launch / steps, keys with and without families: 1 pair 256 x 256 293 / 448 and 459 / 586, 512 x
// 96 382 / 456 and 853 / 787, 64 pairs 512 x 128 1417 / 1489 and 2317 / 2348.  So the lines are safe and no longer where the two ways
// meet; where that is has not been measured.
// More than 512 points always take the steps (refreshes of 64 blocks of 256 .. 1100 points average 1133 us with the line
// at 512 points, 1181 with it at 1024).
constexpr int kLevelMaxPts = 512;
constexpr int kLevelMaxK = 101;          // (the most the lines below admit, with no more clusters than points)
inline bool coarse_level_fits(long long pairs, int max_pts, int max_k)
{
    if (max_pts < 1 || max_k < 1 || max_pts > kLevelMaxPts || max_k > kLevelMaxK) return false;
    if (max_k < 64 || max_pts * max_k <= 10240) return true;
    return max_pts <= 256 && max_k <= (pairs >= 192 ? 96 : pairs >= 32 ? 64 : 0);
}

}  // namespace mp
