// Centroid update of k-means after the first Lloyd iteration (Sec. 3.1: centroid = mean of the members): the member sums
// of the iteration before, moved by the points that changed cluster.
//
// From the second iteration on few points move -- of 16.8 M keys in blocks of 8192 with 256 centroids 20, 8, 5, 2.5, 1.3
// per cent in iterations 2 to 6, half a per cent in the tenth -- while summing afresh reads every key and sorts every
// point into a member list.  The sums have to be those of the definition, which adds a cluster's members in sequence
// order in fp64, rounding after every addition: the two are the same where no addition rounds at all.  All keys of a
// block are multiples of 2^e, e the exponent of the last place of its smallest nonzero element, and below 2^E, so a sum of up to n of
// them is a multiple of 2^e below n 2^E, hence exact in 53 bits whatever its order while n 2^E <= 2^(53 + e).  The first
// iteration notes e and E per cluster; a workgroup that finds a cluster too large for its block's range (or an infinity or
// NaN in the block) sums the clusters that changed afresh, member after member in sequence order, as defined.
//
// A block of which no point moved has the centroids it had, so the next step keeps its assignment without looking at a key
// (refresh of eight 8K contexts 804 -> 744 us).
//
// 2048 blocks of 8192 keys x 256 centroids, iterations 2 to 10: 711, 428, 322, 248, 203, 156, 132, 110, 95 us instead of 970
// (member lists 123, means 846); 32 such blocks: 20 to 10 us instead of 34.  With marks, ranges and counts asked for together instead
// of one after the other, averages of nine iterations: 269 -> 238 and 12.6 -> 12.1 us.
#include "mp_device.h"
#include "mp_internal.h"

namespace mp {

namespace {

constexpr int kMoveWaves = 8;
constexpr int kMoveThreads = 64 * kMoveWaves;
constexpr int kMoveSteps = 6;
constexpr int kMoveRound = kMoveThreads * kMoveSteps;        // points looked at at a time
constexpr int kMoveClusters = 256;                           // most clusters of a workgroup
constexpr int kMoveBatch = 8;                                // rows on their way to sixteen lanes at once
constexpr int kMoveMany = 8 * kMoveBatch;                    // more entries of a cluster than this take a wave
constexpr int kListRoom = 4 * kMoveRound;                    // members listed at a time while sums are taken afresh
constexpr int kListReach = 65536;                            // ... of this many points of the block

// Eight bf16 values to eight sums, in fp64.
__device__ __forceinline__ void add8(double (&a)[8], const uint4& w)
{
    const uint32_t d[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a[2 * i] += (double)bf16lo_to_f32(d[i]);
        a[2 * i + 1] += (double)bf16hi_to_f32(d[i]);
    }
}

// One workgroup per p.per clusters of a (block, unit).  It collects the points that the assignment marked, sorts those that
// left or entered one of its clusters by cluster (in any order inside it), and sixteen lanes a cluster take the rows of
// these points to the stored sum, eight dims each; all four sixteens of a wave share out a cluster of many such points.
// Latency bound: a trip for the marks, one for the points' ids, one for the sum and eight rows, one for every eight rows more
// (or 32); so four clusters to a wave and sixteen waves, two workgroups, to a compute unit (116 registers).  Where one cluster
// takes most of what moves, 8192 keys of which half are zeros in 256 clusters, a build of five iterations: 2789 us with all
// members summed in every iteration, 3480 with eight rows a trip in any case, 2100 so.
// grid = (groups of p.per clusters of a block, blocks, units)
__global__ __launch_bounds__(kMoveThreads, 4) void move_means_kernel(const MoveMeans p)
{
    __shared__ uint32_t points[kMoveRound];                  // of the block
    __shared__ uint32_t entries[2 * kMoveRound];             // point << 1 | it went (one that moves is in two clusters' entries)
    __shared__ int total[kMoveClusters], at[kMoveClusters], due[kMoveClusters];
    __shared__ bool touched[kMoveClusters], fresh[kMoveClusters];
    __shared__ int top, bottom, most, n_marked, n_points, n_few, n_many, held;
    const int b = blockIdx.y, u = blockIdx.z;
    asm volatile("" ::"s"(p.blocks), "s"(p.marks), "s"(p.sum), "s"(p.per));      // (the arguments' lines in one trip)
    typedef const __attribute__((address_space(4))) int32_t constant_int;
    const constant_int* block = (constant_int*)p.blocks + 4 * b;
    const int x0 = block[0], x1 = block[1], k0 = block[2], k1 = block[3];
    const int ka = k0 + (int)blockIdx.x * p.per, m = min(p.per, k1 - ka);
    if (m <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, part = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = x1 - x0, chunks = (n + 63) / 64;
    const unsigned long long* marks = p.marks + u * p.marks_stride + first_mark(x0, b);
    const int32_t* was = p.old_ids + u * p.ids_stride + x0;
    const int32_t* now = p.new_ids + u * p.ids_stride + x0;
    const uint4* Xb = reinterpret_cast<const uint4*>(p.X + ((long long)u * p.x_unit_rows + x0) * kHeadDim) + part;
    int32_t* count = p.count + u * p.count_stride + ka;

    // the first of what every thread looks at, in one trip: the range of a cluster's keys, 64 points' marks, a cluster's members
    const int chunk0 = wave + kMoveWaves * lane;
    const uint32_t range0 = k0 + tid < k1 ? p.range[u * p.range_stride + k0 + tid] : 255u;
    const unsigned long long marks0 = chunk0 < chunks ? marks[chunk0] : 0ull;
    const int count0 = tid < m ? count[tid] : 0;
    if (tid == 0) { top = 0; bottom = 255; most = 0; n_marked = 0; }
    if (tid < m) touched[tid] = fresh[tid] = false;
    __syncthreads();
    {
        // range of the block's keys, marks of the block
        int hi = (int)(range0 >> 16), lo = (int)(range0 & 0xffffu), marked = __popcll(marks0);
        for (int i = k0 + tid + kMoveThreads; i < k1; i += kMoveThreads) {
            const uint32_t r = p.range[u * p.range_stride + i];
            hi = max(hi, (int)(r >> 16));
            lo = min(lo, (int)(r & 0xffffu));
        }
        for (int i = chunk0 + kMoveThreads; i < chunks; i += kMoveThreads) marked += __popcll(marks[i]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            hi = max(hi, __shfl_xor(hi, off, 64));
            lo = min(lo, __shfl_xor(lo, off, 64));
            marked += __shfl_xor(marked, off, 64);
        }
        if (lane == 0) { atomicMax(&top, hi); atomicMin(&bottom, lo); atomicAdd(&n_marked, marked); }
    }
    __syncthreads();
    if (n_marked == 0) return;
    // (a round takes all chunks of 64 points, or as many as its points fit in any case)
    const bool one_round = n_marked <= kMoveRound;
    const int step = one_round ? chunks : kMoveRound / 64;
    // cluster c of this workgroup, the lane's eight dims: its sum, and what goes with it once the sum is final
    auto sum_of = [&](int c) { return reinterpret_cast<double2*>(p.sum + ((long long)u * p.sum_unit_rows + ka + c) * kHeadDim) + 4 * part; };
    auto read_sum = [&](int c, double (&a)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double2 v = sum_of(c)[i];
            a[2 * i] = v.x;
            a[2 * i + 1] = v.y;
        }
    };
    auto store_sum = [&](int c, const double (&a)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sum_of(c)[i] = make_double2(a[2 * i], a[2 * i + 1]);
    };
    // (the row a mean takes the place of is asked for with the sum: the next assignment looks at centroids that changed only)
    auto mean_of = [&](int c) { return reinterpret_cast<uint4*>(p.C + ((long long)u * p.c_unit_rows + ka + c) * kHeadDim) + part; };
    auto store_mean = [&](int c, int members, const double (&a)[8], const uint4& before) {
        if (members == 0) return;                            // (an empty cluster keeps its centroid)
        const double den = (double)members, inv = 1.0 / den;
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = (uint32_t)quotient_to_bf16(a[2 * i], den, inv) | ((uint32_t)quotient_to_bf16(a[2 * i + 1], den, inv) << 16);
        *mean_of(c) = make_uint4(w[0], w[1], w[2], w[3]);
        if (!p.changed) return;
        const unsigned long long differs = __ballot(w[0] != before.x || w[1] != before.y || w[2] != before.z || w[3] != before.w);
        if (part == 0 && ((differs >> (lane & 48)) & 0xffffull) != 0) fresh[c] = true;
    };
    bool exact = true;
    for (int ca = 0; ca < chunks; ca += step) {
        const int cb = min(ca + step, chunks);
        if (tid < m) total[tid] = 0;
        if (tid == 0) n_points = 0;
        __syncthreads();
        for (int c0 = ca + wave; c0 < cb; c0 += kMoveThreads) {      // the marked points, in any order
            const int chunk = c0 + kMoveWaves * lane;
            const unsigned long long mark = chunk >= cb ? 0ull : chunk == chunk0 ? marks0 : marks[chunk];
            const int has = __popcll(mark), incl = (int)wave_incl_scan_u32((uint32_t)has);
            int base = 0;
            if (lane == 63) base = atomicAdd(&n_points, incl);
            base = __builtin_amdgcn_readlane(base, 63);
            for (unsigned long long left = __ballot(has != 0); left != 0; left &= left - 1) {
                const int j = __ffsll((long long)left) - 1;
                const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)mark, j), hi = __builtin_amdgcn_readlane((uint32_t)(mark >> 32), j);
                const int first = base + __builtin_amdgcn_readlane(incl - has, j);
                if ((((unsigned long long)hi << 32 | lo) >> lane) & 1ull)
                    points[first + (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u))] =
                        (uint32_t)((c0 + kMoveWaves * j) * 64 + lane);
            }
        }
        __syncthreads();
        const int n_here = __builtin_amdgcn_readfirstlane(n_points);
        uint32_t o[kMoveSteps], e[kMoveSteps];               // old and new cluster of a point, counted from ka
        // (a lane past the last point reads the first point of the block: under a lane mask each step waits for the one before)
#pragma unroll
        for (int r = 0; r < kMoveSteps; ++r) {
            const int i = r * kMoveThreads + tid;
            o[r] = e[r] = 0u;
            if (r * kMoveThreads < n_here) {
                const uint32_t t = i < n_here ? points[i] : 0u;
                o[r] = (uint32_t)was[t];
                e[r] = (uint32_t)now[t];
            }
        }
#pragma unroll
        for (int r = 0; r < kMoveSteps; ++r) {
            o[r] -= (uint32_t)ka;
            e[r] = r * kMoveThreads + tid < n_here ? e[r] - (uint32_t)ka : o[r];
        }
#pragma unroll
        for (int r = 0; r < kMoveSteps; ++r) {
            if (o[r] == e[r]) continue;
            if (o[r] < (uint32_t)m) atomicAdd(&total[o[r]], 1);
            if (e[r] < (uint32_t)m) atomicAdd(&total[e[r]], 1);
        }
        __syncthreads();
        // the most members any sum on the way can have: those of before and every point that comes
        if (ca == 0 && tid < m && total[tid] != 0) atomicMax(&most, count0 + total[tid]);
        const bool last = cb == chunks;
        // entries of a cluster side by side; the clusters that have any: those with few of them from the front, the others from the back
        if (wave == 0) {
            int entry = 0, few = 0, many = 0;
            for (int c = lane; c - lane < m; c += 64) {
                const int mine = c < m ? total[c] : 0;
                const int incl = (int)wave_incl_scan_u32((uint32_t)mine);
                const bool is_due = mine != 0 || (last && c < m && touched[c]);
                const unsigned long long f = __ballot(is_due && mine <= kMoveMany), g = __ballot(mine > kMoveMany);
                auto before = [](unsigned long long x) { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(x >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)x, 0u)); };
                if (c < m) at[c] = entry + incl - mine;
                if (is_due) due[mine <= kMoveMany ? few + before(f) : kMoveClusters - 1 - many - before(g)] = c;
                entry += __builtin_amdgcn_readlane(incl, 63);
                few += __popcll(f);
                many += __popcll(g);
            }
            if (lane == 0) { n_few = few; n_many = many; }
        }
        __syncthreads();
        if (tid == 0 && n_few + n_many > 0) p.moved[u * p.moved_stride + b] = 1;
        if (ca == 0) {
            const int room = 45 - (top - bottom);            // 53 + e - E in terms of the exponent fields
            const int members = one_round ? most : n;
            exact = top < 255 && room >= 0 && members <= (1 << min(room, 30));
            if (!exact) {
                // (the points of later rounds are not looked at: one of them may have moved)
                if (!one_round && tid == 0) p.moved[u * p.moved_stride + b] = 1;
                break;
            }
        }
#pragma unroll
        for (int r = 0; r < kMoveSteps; ++r) {
            if (o[r] == e[r]) continue;
            const uint32_t i = points[r * kMoveThreads + tid] << 1;
            if (o[r] < (uint32_t)m) entries[atomicAdd(&at[o[r]], 1)] = i | 1u;
            if (e[r] < (uint32_t)m) entries[atomicAdd(&at[e[r]], 1)] = i;
        }
        __syncthreads();
        // entries [i0, i0 + kMoveBatch) from `first`, as far as there are `all`, to the sum; returns how many of them went
        auto take = [&](double (&a)[8], int first, int i0, int all) {
            uint4 w[kMoveBatch];
            int gone = 0;
#pragma unroll
            for (int q = 0; q < kMoveBatch; ++q) {
                const int i = i0 + q;
                const uint32_t e = entries[first + min(i, all - 1)];
                w[q] = Xb[(long long)(e >> 1) * 16];
                const uint32_t keep = i < all ? ~0u : 0u, turn = e & 1u ? 0x80008000u & keep : 0u;
                gone += turn != 0u ? 1 : 0;
                w[q] = make_uint4((w[q].x & keep) ^ turn, (w[q].y & keep) ^ turn, (w[q].z & keep) ^ turn, (w[q].w & keep) ^ turn);
            }
#pragma unroll
            for (int q = 0; q < kMoveBatch; ++q) add8(a, w[q]);
            return gone;
        };
        auto store = [&](int c, int due_here, int gone, const double (&a)[8], const uint4& before) {
            if (due_here != 0) store_sum(c, a);
            const int members_now = count[c] + due_here - 2 * gone;
            if (part == 0) {
                count[c] = members_now;
                touched[c] = true;
            }
            if (last) store_mean(c, members_now, a, before);
        };
        // a cluster of many entries: every sixteen lanes of a wave take a quarter of them
        for (int d = wave; d < n_many; d += kMoveWaves) {
            const int c = due[kMoveClusters - 1 - d], due_here = total[c], first = at[c] - due_here;
            double a[8] = {};
            uint4 before = make_uint4(0, 0, 0, 0);
            if (lane < 16) {
                read_sum(c, a);
                if (p.changed) before = *mean_of(c);
            }
            int gone = 0;
            for (int i0 = kMoveBatch * (lane >> 4); i0 < due_here; i0 += 4 * kMoveBatch) gone += take(a, first, i0, due_here);
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) {
#pragma unroll
                for (int i = 0; i < 8; ++i) a[i] += __shfl_xor(a[i], off, 64);
                gone += __shfl_xor(gone, off, 64);
            }
            if (lane < 16) store(c, due_here, gone, a, before);
        }
        for (int d0 = 4 * wave; d0 < n_few; d0 += 4 * kMoveWaves) {
            const int d = d0 + (lane >> 4);
            if (d >= n_few) continue;
            const int c = due[d], due_here = total[c], first = at[c] - due_here;
            double a[8];
            read_sum(c, a);
            uint4 before = make_uint4(0, 0, 0, 0);
            if (p.changed) before = *mean_of(c);
            int gone = 0;
            for (int i0 = 0; i0 < due_here; i0 += kMoveBatch) gone += take(a, first, i0, due_here);
            store(c, due_here, gone, a, before);
        }
        __syncthreads();
    }
    auto say_changed = [&] { if (p.changed && tid < m) p.changed[u * p.range_stride + ka + tid] = fresh[tid] ? 1u : 0u; };
    if (exact) {
        say_changed();
        return;
    }

    // ---- the sums round: members one after the other, in sequence order, of every cluster that changed (as far as the
    // first round of moves tells; all of them where there are more).  A stable sort of a segment's points by cluster, each
    // wave an eighth of them (as in block_lists_kernel), then a wave a cluster, 32 rows at a time.  Keys of which a tenth is
    // 1e-12 times the others, builds with lists and sums of all members in every iteration -> here: 32 blocks of 8192 keys, ten
    // iterations 1350 -> 1219 us, 512 blocks 7164 -> 6865; 64 blocks of 2000 keys, five iterations 433 -> 399. ----
    static_assert(kListRoom * 2 <= (int)sizeof(entries) && kMoveWaves * kMoveClusters * 4 <= (int)sizeof(points), "");
    uint16_t* list = reinterpret_cast<uint16_t*>(entries);
    int* place = reinterpret_cast<int*>(points);             // [kMoveWaves][m]
    const int thirds = m > 1 ? (32 - __clz(m - 1) + 2) / 3 : 0;
    // (the members its clusters had and every point that may have come: with few clusters of a long block they fit the list)
    if (tid == 0) held = n_marked;
    __syncthreads();
    if (tid < m) atomicAdd(&held, count0);
    __syncthreads();
    const int segment = held <= kListRoom ? kListReach : kListRoom;
    for (int s0 = 0; s0 < n; s0 += segment) {
        const int here = min(segment, n - s0);
        const int per_wave = (here + kMoveThreads - 1) / kMoveThreads * 64, t0 = s0 + min(wave * per_wave, here), t1 = s0 + min((wave + 1) * per_wave, here);
        int* mine = place + wave * m;
        __syncthreads();
        for (int i = tid; i < kMoveWaves * m; i += kMoveThreads) place[i] = 0;
        __syncthreads();
        // the wave's points in order, 64 at a time: their clusters, counted from ka
        auto walk = [&](auto use) {
            constexpr int kAhead = 16;                       // ids on their way at once
            for (int tb = t0; tb < t1; tb += 64 * kAhead) {
                int id[kAhead];
#pragma unroll
                for (int r = 0; r < kAhead; ++r) id[r] = now[min(tb + 64 * r + lane, t1 - 1)] - ka;
#pragma unroll
                for (int r = 0; r < kAhead; ++r) {
                    const int t = tb + 64 * r + lane;
                    use(t - s0, id[r], t < t1 && (unsigned)id[r] < (unsigned)m);
                }
            }
        };
        walk([&](int, int id, bool valid) { if (valid) atomicAdd(&mine[id], 1); });
        __syncthreads();
        for (int c = tid; c < m; c += kMoveThreads) {
            int all = 0;
            for (int w = 0; w < kMoveWaves; ++w) all += place[w * m + c];
            at[c] = all;
        }
        __syncthreads();
        if (wave == 0) {                                     // at: members in this segment -> first place
            int first = 0;
            for (int c = lane; c - lane < m; c += 64) {
                const int all = c < m ? at[c] : 0, incl = (int)wave_incl_scan_u32((uint32_t)all);
                if (c < m) at[c] = first + incl - all;
                first += __builtin_amdgcn_readlane(incl, 63);
            }
        }
        __syncthreads();
        for (int c = tid; c < m; c += kMoveThreads) {
            int next = at[c];
            for (int w = 0; w < kMoveWaves; ++w) {
                const int some = place[w * m + c];
                place[w * m + c] = next;
                next += some;
            }
        }
        __syncthreads();
        walk([&](int t, int id, bool valid) {
            if (!__any(valid)) return;
            const unsigned long long same = lanes_with_id(id, valid, thirds);
            const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            if (valid) {
                const int first = mine[id];
                list[first + rank] = (uint16_t)t;
                if (rank == 0) mine[id] = first + __popcll(same);
            }
        });
        __syncthreads();
        const uint32_t* Xs = reinterpret_cast<const uint32_t*>(Xb - part) + (long long)s0 * (kHeadDim / 2) + lane;
        const int n_sums = one_round ? n_few + n_many : m;
        for (int d = wave; d < n_sums; d += kMoveWaves) {    // (a lane has two dims, as in cluster_mean_kernel)
            const int c = !one_round ? d : d < n_few ? due[d] : due[kMoveClusters - 1 - (d - n_few)];
            const int first = at[c], end = place[(kMoveWaves - 1) * m + c];
            double2* sum = reinterpret_cast<double2*>(p.sum + ((long long)u * p.sum_unit_rows + ka + c) * kHeadDim) + lane;
            double2 a = make_double2(0.0, 0.0);
            int members = end - first;
            if (s0 > 0) {
                a = *sum;
                members += count[c];
            }
            for (int base = first; base < end; base += 64) {
                const int here_now = min(end - base, 64), member = lane < here_now ? list[base + lane] : 0;
                constexpr int kBatch = 32;
                for (int q0 = 0; q0 < here_now; q0 += kBatch) {
                    uint32_t w[kBatch];
#pragma unroll
                    for (int q = 0; q < kBatch; ++q) w[q] = Xs[(long long)__builtin_amdgcn_readlane(member, min(q0 + q, here_now - 1)) * (kHeadDim / 2)];
#pragma unroll
                    for (int q = 0; q < kBatch; ++q) {
                        if (q0 + q < here_now) {
                            a.x += (double)bf16lo_to_f32(w[q]);
                            a.y += (double)bf16hi_to_f32(w[q]);
                        }
                    }
                }
            }
            *sum = a;
            if (lane == 0) count[c] = members;
            if (s0 + segment >= n && members > 0) {     // (an empty cluster keeps its centroid)
                const double den = (double)members, inv = 1.0 / den;
                uint32_t* row = reinterpret_cast<uint32_t*>(p.C + ((long long)u * p.c_unit_rows + ka + c) * kHeadDim) + lane;
                const uint32_t w = (uint32_t)quotient_to_bf16(a.x, den, inv) | ((uint32_t)quotient_to_bf16(a.y, den, inv) << 16);
                const bool differs = p.changed && __any(w != *row);
                *row = w;
                if (lane == 0 && differs) fresh[c] = true;
            }
        }
    }
    __syncthreads();
    say_changed();
}

}  // namespace

hipError_t launch_move_means(MoveMeans p, int nb, int max_k, int U, hipStream_t s)
{
    if (nb <= 0 || max_k <= 0 || U <= 0) return hipSuccess;
    // two workgroups a compute unit, sixteen to 256 clusters each
    const long long pairs = (long long)nb * U;
    const long long want = (512 + pairs - 1) / pairs;
    p.per = (int)((max_k + want - 1) / want);
    p.per = p.per < 16 ? 16 : p.per > kMoveClusters ? kMoveClusters : p.per;
    hipLaunchKernelGGL(move_means_kernel, dim3((max_k + p.per - 1) / p.per, nb, U), dim3(kMoveThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace mp
