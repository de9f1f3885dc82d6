// Sizes that the value pass's launch is planned with: plain host functions of the call's sizes, so that they can be checked
// without a GPU.
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
// are not (some then have two, and these are the call's time).  So: as many per unit as fit one round, if that fills two
// thirds of it, else as many as fit two (both resident at once).  Dense, 32768 rows, 4 heads, us by workgroups per unit:
// 86 units 2: 222, 3: 305, 5: 214; 96: 2: 243, 3: 314, 4: 252; 129: 1: 389, 2: 461, 3: 330; 144: 1: 398, 2: 465, 3: 353;
// 160: 1: 415, 2: 486, 3: 392; 176: 1: 438, 2: 508; 192: 1: 476, 2: 509.
// More units than compute units: the count (of up to six rounds) whose last round is fullest; 264 units 1: 883, 2: 756,
// 3: 714, 5: 707; 320: 2: 793, 3: 778, 4: 816.
constexpr int kStreamWgs = 256;
inline int stream_chunks_per_unit(int n_units)
{
    if (n_units <= kStreamWgs) {
        const int one = kStreamWgs / n_units;
        return 3 * one * n_units >= 2 * kStreamWgs ? one : 2 * kStreamWgs / n_units;
    }
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

// Rows per chunk when n rows are cut into at most `chunks` chunks of about the same size: a multiple of 64 (16 rows a wave
// and tile).
inline int stream_chunk_rows(long long n, int chunks)
{
    const long long per = (n + chunks - 1) / chunks;
    return (int)std::max<long long>(64, (per + 63) / 64 * 64);
}

// Rows per chunk of the selected keys (or centroid terms) and of the tail.  Chunks of both are about the same length, in
// all one more than the count above at most: a short tail is one short chunk and takes none away from the keys.  (It took
// one of two from units 86 to 128, and both streams had one chunk each: 96 units, 2048 keys, tail of 130, 4 heads, whole
// step 57 us, now 42.)  Each stream's chunks are cut evenly, so that a short one's rows are spread over its four waves.
struct StreamPlan {
    int first_rows, tail_rows;
};
inline StreamPlan plan_streams(int n_units, long long first, long long tail)
{
    const int rows = stream_chunk_rows(first + tail, stream_chunks_per_unit(n_units));
    auto even = [&](long long n) { return stream_chunk_rows(n, (int)std::max<long long>(1, (n + rows - 1) / rows)); };
    return StreamPlan{even(first), even(tail)};
}

}  // namespace mp
