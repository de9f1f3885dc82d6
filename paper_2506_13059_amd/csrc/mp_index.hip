// Index construction kernels for gfx950: member lists (stable counting sort by cluster id),
// cluster-contiguous gather of the KV rows, and the per-cluster tables (N, key centroid, value
// centroid = bf16-rounded fp64 means of the member keys / values, Sec. 3.1 and 3.2).
//
// Member sums run over the members in sequence order, one wave per cluster, in fp64: the result
// does not depend on the launch shape and repeats bit for bit.
#include <algorithm>
#include <type_traits>

#include "mp_device.h"
#include "mp_internal.h"

namespace mp {

namespace {

// Member lists and their offsets for every block of a unit in one launch: a stable counting sort of
// the block's points by cluster id.  One workgroup of 16 waves per (block, unit); `waves` of them
// walk one contiguous segment of the block's points each, 64 points at a time.
//   Among the 64 points of a step, the lanes that share this lane's id are found with one ballot per
//   id bit; a point's rank among them is the number of such lanes below it, and the lowest of them
//   adds their number to the segment's counter of that id (LDS, touched by this wave only).
//   walk 1 counts; then counter[w][id] becomes the position of the first member of id in segment w
//   (block offset + exclusive prefix over ids + members in earlier segments); walk 2 writes the
//   members at counter + rank.  Within a cluster the members end up in ascending point order.
// Bound by the instructions of the one workgroup (a 64-point step is some fifty, four waves share a SIMD) and by its
// trips to memory and LDS in a row.  So a segment of up to sixteen steps (blocks of up to 16384 points, where the
// counters leave room for sixteen waves) is loaded at once and ranked once: a lane keeps its points' ids and their ranks
// in the segment's cluster, and walk 2 is a read and a write.  Longer segments are walked twice.  32 blocks of 8192
// points, 256 clusters each: 17.3 -> 13.6 us a launch; 64 of 8219 points, 273 clusters: 24.7 -> 13 us.
// start[u][id] = first list position of cluster id (positions count from the first point of the
// launch, `p_first`); the last block also writes the end position after its last cluster.
// Dynamic LDS: (waves + 1) * max clusters per block int32.
constexpr int kListWaves = 16;
constexpr int kListSteps = 16;

__global__ __launch_bounds__(1024) void block_lists_kernel(const int32_t* __restrict__ ids, long long ids_stride,
                                                           const int32_t* __restrict__ blocks /*[nb][4]: x0,x1,k0,k1*/,
                                                           int p_first, int waves, int32_t* __restrict__ start,
                                                           long long start_stride, int32_t* __restrict__ list,
                                                           long long list_stride)
{
    extern __shared__ int32_t lists_lds[];
    __shared__ int32_t wave_tot[kListWaves];
    const int b = blockIdx.x, u = blockIdx.y;
    const int x0 = blocks[4 * b + 0], x1 = blocks[4 * b + 1], k0 = blocks[4 * b + 2], k1 = blocks[4 * b + 3];
    const int k = k1 - k0, n = x1 - x0;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int32_t* ctr = lists_lds;                  // [waves][k]
    int32_t* tot = lists_lds + waves * k;      // [k]
    const int32_t* idp = ids + u * ids_stride;
    int32_t* lp = list + u * list_stride;
    const int thirds = k > 1 ? (32 - __clz(k - 1) + 2) / 3 : 0;
    const int seg = (((n + waves - 1) / waves) + 63) & ~63;
    const int s0 = x0 + wave * seg, s1 = (s0 + seg < x1) ? s0 + seg : x1;
    const bool keep = seg <= 64 * kListSteps;
    int32_t* my = ctr + wave * k;
    uint32_t kept[kListSteps];                 // rank in the segment's cluster << 16 | id (at most 8192 clusters a block)

    if (keep && wave < waves) {
#pragma unroll
        for (int r = 0; r < kListSteps; ++r) {
            const int t = s0 + 64 * r + lane;
            kept[r] = t < s1 ? (uint32_t)(idp[t] - k0) : 0u;
        }
    }
    for (int i = tid; i < waves * k; i += 1024) ctr[i] = 0;
    __syncthreads();
    // 64 points: the rank of each among the points of its cluster that this wave has seen since the counter's start
    auto rank_step = [&](int id, bool valid) {
        const unsigned long long same = lanes_with_id(id, valid, thirds);
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        int at = 0;
        if (valid) {
            at = my[id] + rank;
            if (rank == 0) my[id] = at + __popcll(same);
        }
        return at;
    };
    // one walk over the wave's segment; kWrite = false: count, true: place
    auto walk = [&](auto write_tag) {
        constexpr bool kWrite = decltype(write_tag)::value;
        if (wave >= waves) return;
        for (int t0 = s0; t0 < s1; t0 += 256) {
            int id4[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = t0 + 64 * r + lane;
                id4[r] = t < s1 ? idp[t] - k0 : 0;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = t0 + 64 * r + lane;
                const int at = rank_step(id4[r], t < s1);
                if (kWrite && t < s1) lp[at] = t;
            }
        }
    };
    if (keep) {
        if (wave < waves) {
#pragma unroll
            for (int r = 0; r < kListSteps; ++r)
                if (s0 + 64 * r < s1) kept[r] |= (uint32_t)rank_step((int)kept[r], s0 + 64 * r + lane < s1) << 16;
        }
    } else {
        walk(std::false_type{});
    }
    __syncthreads();
    // counts per segment -> first positions: totals per id, exclusive prefix over ids, segments in order
    const int per = (k + 1023) / 1024;          // consecutive ids per thread
    const int i0 = tid * per, i1 = (i0 + per < k) ? i0 + per : k;
    const bool in_registers = per == 1 && waves == kListWaves;
    int counts[kListWaves];
    int run = 0;
    if (in_registers) {
#pragma unroll
        for (int w = 0; w < kListWaves; ++w) counts[w] = i0 < k ? ctr[w * k + i0] : 0;
#pragma unroll
        for (int w = 0; w < kListWaves; ++w) run += counts[w];
    } else {
        for (int id = i0; id < i1; ++id) {
            int c = 0;
            for (int w = 0; w < waves; ++w) c += ctr[w * k + id];
            tot[id] = c;
            run += c;
        }
    }
    const int incl = (int)wave_incl_scan_u32((uint32_t)run);
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int pos = x0 - p_first + incl - run;
    for (int w = 0; w < wave; ++w) pos += wave_tot[w];
    if (in_registers) {
        if (i0 < k) {
            start[u * start_stride + k0 + i0] = pos;
#pragma unroll
            for (int w = 0; w < kListWaves; ++w) {
                ctr[w * k + i0] = pos;
                pos += counts[w];
            }
        }
    } else {
        for (int id = i0; id < i1; ++id) {
            start[u * start_stride + k0 + id] = pos;
            int q = pos;
            for (int w = 0; w < waves; ++w) {
                const int c = ctr[w * k + id];
                ctr[w * k + id] = q;
                q += c;
            }
            pos += tot[id];
        }
    }
    if (b == (int)gridDim.x - 1 && tid == 0) start[u * start_stride + k1] = x1 - p_first;
    __syncthreads();
    if (keep) {
        if (wave < waves) {
#pragma unroll
            for (int r = 0; r < kListSteps; ++r) {
                const int t = s0 + 64 * r + lane;
                if (t < s1) lp[my[kept[r] & 0xffffu] + (int)(kept[r] >> 16)] = t;
            }
        }
    } else {
        walk(std::true_type{});
    }
}

// Where the gather leaves rows s >= t0 of its sources once more, in sequence order: row s - t0 of K and V (each optional).
__device__ __forceinline__ void keep_in_sequence(const SequenceCopy& q, int u, long long s, int c, const uint4& k, const uint4& v)
{
    if (s < q.t0) return;
    const long long at = ((long long)u * q.unit_rows + s - q.t0) * 16 + c;
    if (q.K) store_once(reinterpret_cast<uint4*>(q.K) + at, k);
    if (q.V) store_once(reinterpret_cast<uint4*>(q.V) + at, v);
}

// The gather into 8-bit storage.  A value row becomes 128 e4m3 codes (OCP format: bias 7,
// largest magnitude 448, no infinities) and one fp32 scale, scale = max|x| / 448 (1 for a zero row),
// code = x / scale rounded to nearest even; both divisions are IEEE fp32.  A key row is stored the
// same way as its residual from the key centroid of its fine cluster, x = fp32(k) - fp32(centroid):
// the decode step already has q . centroid, and the residual is small where the key itself is not.
// Sixteen threads share a row (8 elements of the key and 8 of the value each);
// scales[u][row] = {key scale, value scale}.
// Elementwise fp32 difference of two groups of eight bf16 values.
struct F8 { float v[8]; };
__device__ __forceinline__ F8 widen8(const uint4& w)
{
    const uint32_t d[4] = {w.x, w.y, w.z, w.w};
    F8 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o.v[2 * i] = bf16lo_to_f32(d[i]);
        o.v[2 * i + 1] = bf16hi_to_f32(d[i]);
    }
    return o;
}
__device__ __forceinline__ float absmax8(const F8& x)
{
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) a = fmaxf(a, fabsf(x.v[i]));
    return a;
}
__device__ __forceinline__ uint2 e4m3_codes8(const F8& x, float scale)
{
    // (the quotient of the row's largest entry may exceed 448 by an ulp: clamp, so that the conversion never overflows)
    auto q = [&](float v) { return fminf(fmaxf(v / scale, -448.f), 448.f); };
    int out[2] = {0, 0};
    out[0] = __builtin_amdgcn_cvt_pk_fp8_f32(q(x.v[0]), q(x.v[1]), out[0], false);
    out[0] = __builtin_amdgcn_cvt_pk_fp8_f32(q(x.v[2]), q(x.v[3]), out[0], true);
    out[1] = __builtin_amdgcn_cvt_pk_fp8_f32(q(x.v[4]), q(x.v[5]), out[1], false);
    out[1] = __builtin_amdgcn_cvt_pk_fp8_f32(q(x.v[6]), q(x.v[7]), out[1], true);
    return make_uint2((uint32_t)out[0], (uint32_t)out[1]);
}
__global__ void gather_quantize_rows_kernel(const uint4* __restrict__ srcK, const uint4* __restrict__ srcV,
                                            long long src_unit_rows, const int32_t* __restrict__ list,
                                            long long list_stride, const int32_t* __restrict__ ids, long long ids_stride,
                                            const uint4* __restrict__ Kc, long long kc_unit_rows, int n,
                                            uint2* __restrict__ dstK, uint2* __restrict__ dstV,
                                            float2* __restrict__ scales, long long dst_unit_rows, int dst_row0,
                                            const SequenceCopy seq, int32_t* __restrict__ unusual)
{
    const int u = blockIdx.y;
    const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long p = g >> 4;
    const int c = (int)(g & 15);
    if (p >= n) return;   // (all sixteen threads of a row leave together)
    const long long s = list[u * list_stride + p];
    const long long f = ids[u * ids_stride + s];
    const uint4 kw = srcK[((long long)u * src_unit_rows + s) * 16 + c], vw = srcV[((long long)u * src_unit_rows + s) * 16 + c];
    keep_in_sequence(seq, u, s, c, kw, vw);
    F8 k = widen8(kw);
    const F8 cen = widen8(Kc[((long long)u * kc_unit_rows + f) * 16 + c]);
    const F8 v = widen8(vw);
#pragma unroll
    for (int i = 0; i < 8; ++i) k.v[i] -= cen.v[i];
    float ka = absmax8(k), va = absmax8(v);
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        ka = fmaxf(ka, __shfl_xor(ka, off, 64));
        va = fmaxf(va, __shfl_xor(va, off, 64));
    }
    const float ks = ka > 0.f ? ka / 448.f : 1.f, vs = va > 0.f ? va / 448.f : 1.f;
    const long long row = (long long)u * dst_unit_rows + dst_row0 + p;
    dstK[row * 16 + c] = e4m3_codes8(k, ks);
    dstV[row * 16 + c] = e4m3_codes8(v, vs);
    if (c == 0) {
        scales[row] = make_float2(ks, vs);
        if (!(vs >= kSmallScale && vs < kLargeScale)) *unusual = 1;
    }
}

// The fp64 sum of rows lp[s0 .. s1) (no list: s0 .. s1) of Xu in that order, by one wave: lane l has dims 2l and 2l+1.
// passes(at, q, row, w) is told every row: it is number at + q of the list, and w the lane's dword of it.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
struct RowSum {
    double a0 = 0.0, a1 = 0.0;
    u16x2 largest = {0, 0}, smallest = {0xffff, 0xffff};     // kRange: magnitudes, and nonzero magnitudes less one
};
template <bool kRange, int kFew, typename Passes>
__device__ __forceinline__ RowSum sum_of_rows(const uint32_t* __restrict__ Xu, const int32_t* __restrict__ lp, int s0, int s1, Passes passes)
{
    const int lane = threadIdx.x & 63;
    RowSum a;
    // 64 member indices at a time (one per lane), then their rows kBatch at a time: the row numbers
    // reach every lane through a lane broadcast, so that kBatch row loads are in flight at once while
    // the additions keep the members' order (a wave's time is the number of trips to memory it makes:
    // with 8 rows a trip the means of coarse clusters of some hundred rows took 160 us per call in an
    // online refresh, with 32 rows a trip a third of that).  The next 64 indices are asked for ahead, and a whole batch has no
    // branch in front of each row: noting the range had made a cluster of thousands 12 % slower (eight blocks of 131072 keys, the
    // longest of 128 clusters, 2009 -> 2254 us); their build, five iterations, 4620 -> 3655 us, of 32 blocks of 8192 keys 828 -> 796.
    // (Zeros in the place of the rows past the end, instead of the branches: one cluster of 8192 350 -> 450 us.)  kFew: up to so many rows
    // are a batch of that size, which jumps over that many places instead of all of them.
    constexpr int kBatch = 32;
    auto members = [&](int base) { return base + lane < s1 ? (lp ? lp[base + lane] : base + lane) : 0; };
    int next = members(s0);
    for (int base = s0; base < s1; base += 64) {
        const int nm = (s1 - base < 64) ? s1 - base : 64;
        const int mine = next;
        if (base + 64 < s1) next = members(base + 64);       // (arrives while these rows travel)
        auto batch = [&](int m, auto full, auto most) {
            constexpr int kMost = decltype(most)::value;
            uint32_t w[kMost];
#pragma unroll
            for (int q = 0; q < kMost; ++q) {
                const long long r = __builtin_amdgcn_readlane(mine, (m + q) & 63);
                w[q] = (full || m + q < nm) ? load_once(&Xu[r * 64 + lane]) : 0u;
            }
#pragma unroll
            for (int q = 0; q < kMost; ++q) {
                if (full || m + q < nm) {
                    passes(base + m, q, __builtin_amdgcn_readlane(mine, (m + q) & 63), w[q]);
                    a.a0 += (double)bf16lo_to_f32(w[q]);
                    a.a1 += (double)bf16hi_to_f32(w[q]);
                    if constexpr (kRange) {
                        const u16x2 size = __builtin_bit_cast(u16x2, w[q] & 0x7fff7fffu);
                        a.largest = __builtin_elementwise_max(a.largest, size);
                        a.smallest = __builtin_elementwise_min(a.smallest, (u16x2)(size - (unsigned short)1));     // (zero: the largest number)
                    }
                }
            }
        };
        for (int m = 0; m < nm; m += kBatch) {
            if (nm - m >= kBatch) batch(m, std::true_type{}, std::integral_constant<int, kBatch>{});
            else if (kFew > 0 && nm - m <= kFew) batch(m, std::false_type{}, std::integral_constant<int, std::max(kFew, 1)>{});
            else batch(m, std::false_type{}, std::integral_constant<int, kBatch>{});
        }
    }
    return a;
}

// Both dims of a lane: the sum over n rows (n > 0) divided once, rounded once to bf16.
__device__ __forceinline__ uint32_t mean_dword(const RowSum& a, int n)
{
    const double den = (double)n;
    return (uint32_t)f64_to_bf16_rne(a.a0 / den) | ((uint32_t)f64_to_bf16_rne(a.a1 / den) << 16);
}

// i modulo n, without the division where i is less than 2 n (it was about one per cent of a call over clusters of a few rows: 158 units of 999
// clusters, 8-bit rows, 411 -> 408 us).
__device__ __forceinline__ unsigned wrapped(unsigned i, unsigned n)
{
    if (i >= n) i -= n;
    if (i >= n) i %= n;
    return i;
}

// One wave per cluster of [k0, k): fp64 sum of the member rows in list order, mean rounded once to bf16.
// Lane l owns dims 2l and 2l+1.  Empty cluster: `fallback` row if given (else zeros).
// mean_out row index = out_row0 + cluster id.  count_out optional.
template <bool kRange>
__global__ __launch_bounds__(256) void cluster_mean_kernel(const uint16_t* __restrict__ X, long long x_unit_rows,
                                                           const int32_t* __restrict__ list, long long list_stride,
                                                           const int32_t* __restrict__ start, long long start_stride,
                                                           int k0, int k, uint16_t* __restrict__ mean_out,
                                                           long long out_unit_rows, int out_row0,
                                                           const uint16_t* __restrict__ fallback,
                                                           long long fb_unit_rows, int32_t* __restrict__ count_out,
                                                           long long count_stride, int count_off,
                                                           double* __restrict__ sum_out, long long sum_unit_rows,
                                                           uint32_t* __restrict__ range_out, uint32_t* __restrict__ changed_out)
{
    const int u = blockIdx.y;
    // (units start at different clusters: workgroups 8 apart share an L2 slice, and the same cluster's of all units would meet there.
    // 64 units of 8192 equal keys, five iterations: 8886 -> 8453 us)
    const int f = k0 + (int)wrapped(blockIdx.x + (unsigned)u, gridDim.x) * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (f >= k) return;
    const int s0 = start[u * start_stride + f], s1 = start[u * start_stride + f + 1];
    const uint32_t* Xu = reinterpret_cast<const uint32_t*>(X + (long long)u * x_unit_rows * kHeadDim);
    const int32_t* lp = list ? list + u * list_stride : nullptr;
    const RowSum a = sum_of_rows<kRange, 0>(Xu, lp, s0, s1, [](int, int, int, uint32_t) {});
    if constexpr (kRange) {
        int hi = max((int)a.largest.x, (int)a.largest.y) >> 7, lo = min((int)a.smallest.x, (int)a.smallest.y);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            hi = max(hi, __shfl_xor(hi, off, 64));
            lo = min(lo, __shfl_xor(lo, off, 64));
        }
        lo = min(max((lo + 1) >> 7, 1), 255);
        if (lane == 0) range_out[u * sum_unit_rows + f] = (uint32_t)hi << 16 | (uint32_t)lo;
    }
    const int n = s1 - s0;
    uint32_t outw;
    if (n > 0) {
        outw = mean_dword(a, n);
    } else if (fallback) {
        outw = reinterpret_cast<const uint32_t*>(fallback + ((long long)u * fb_unit_rows + f) * kHeadDim)[lane];
    } else {
        outw = 0u;
    }
    uint32_t* row = reinterpret_cast<uint32_t*>(mean_out + ((long long)u * out_unit_rows + out_row0 + f) * kHeadDim) + lane;
    if constexpr (kRange) {
        if (changed_out) {                                   // (centroids that an iteration replaces)
            const bool differs = __any(*row != outw);
            if (lane == 0) changed_out[u * sum_unit_rows + f] = differs ? 1u : 0u;
        }
    }
    *row = outw;
    if (count_out && lane == 0) count_out[u * count_stride + count_off + f] = n;
    if (sum_out) reinterpret_cast<double2*>(sum_out + ((long long)u * sum_unit_rows + f) * kHeadDim)[lane] = make_double2(a.a0, a.a1);
}

// Rows list[p0 .. min(p0 + kRows, end)) of X to places p0 ... of `to`, and those from row t0 on to `kept`, by one wave; sixteen
// lanes a row.
template <int kRows>
struct RowMove {
    int place, mine;
    uint4 w[kRows / 4];
    __device__ __forceinline__ void ask_members(const int32_t* __restrict__ list, int p0, int end)
    {
        place = p0;
        mine = list[min(p0 + (int)(threadIdx.x & (kRows - 1)), end - 1)];
    }
    __device__ __forceinline__ int row(int i) const { return __shfl(mine, 4 * i + (int)((threadIdx.x & 63) >> 4), 64); }
    __device__ __forceinline__ void ask_rows(const uint4* __restrict__ X)
    {
#pragma unroll
        for (int i = 0; i < kRows / 4; ++i) w[i] = load_once(X + (long long)row(i) * 16 + (threadIdx.x & 15));
    }
    __device__ __forceinline__ void store(int end, uint4* __restrict__ to, uint4* __restrict__ kept, int t0) const
    {
        const int c = threadIdx.x & 15;
#pragma unroll
        for (int i = 0; i < kRows / 4; ++i) {
            const int at = place + 4 * i + (int)((threadIdx.x & 63) >> 4), r = row(i);
            if (at < end) {
                store_once(to + (long long)at * 16 + c, w[i]);
                if (kept && r >= t0) store_once(kept + (long long)(r - t0) * 16 + c, w[i]);
            }
        }
    }
};
constexpr int kMoveRows = 32;

// Rows to their stored places and the means of the values' clusters in one launch (bf16 storage).  One wave a cluster reads its
// members once, stores them side by side and sums them as cluster_mean_kernel does; keys the same way where their means are
// wanted too (p.key_means), else kMoveRows rows a wave by their places, in the workgroups behind those of the clusters.  Bound by
// memory where the waves fill the chip: refresh of eight 8K contexts 626 -> 552 us (gather, key and value means were a launch each: 178 -> 125 us), build
// of sixteen 128K prompts 20.30 -> 19.67 ms, resumed generation 1227 -> 1144 us.
// A long cluster's sum is a chain of trips to memory, so its rows are moved by whichever of the workgroup's waves are done with theirs.
// Where clusters have a row or two a wave is little more than its start and end: a workgroup without a long cluster has no barrier, and
// few rows are a batch of four.  Tables of keys and values given their clustering, two levels, 64 units of 8192 rows and as many clusters
// 1330 -> 1192 us, with the sums past the caches 1168; 4096 clusters 739 -> 681 -> 660, 2048 392 -> 380 (a launch each for rows and means 1128,
// 661, 408: only where most clusters have a single row, and sums, is that still the shorter way, by 2 to 4 %).
// kSumsOnce: the sums go past the caches (kCachedSums).
template <bool kSumsOnce>
__global__ __launch_bounds__(256) void stored_rows_kernel(const StoredRows p)
{
    __shared__ int ticket[4];
    const int u = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_table = (p.f1 - p.f0 + 3) / 4, of_clusters = p.key_means ? 2 * per_table : per_table;
    const int32_t* list = p.list + u * p.list_stride;
    const bool by_place = (int)blockIdx.x >= of_clusters;
    const int places = (p.n + 4 * kMoveRows - 1) / (4 * kMoveRows), group = (int)blockIdx.x - (by_place ? of_clusters : 0);
    const bool keys = by_place ? group < places : group >= per_table;
    const uint4* X = reinterpret_cast<const uint4*>(keys ? p.K : p.V) + (long long)u * p.src_unit_rows * 16;
    uint4* to = reinterpret_cast<uint4*>(keys ? p.dstK : p.dstV) + ((long long)u * p.dst_unit_rows + p.dst_row0) * 16;
    uint4* kept = reinterpret_cast<uint4*>(keys ? p.seq.K : p.seq.V);
    if (kept) kept += (long long)u * p.seq.unit_rows * 16;
    if (by_place) {
        const int p0 = ((keys ? group : group - places) * 4 + wave) * kMoveRows;
        if (p0 >= p.n) return;
        RowMove<kMoveRows> m;
        m.ask_members(list, p0, p.n);
        m.ask_rows(X);
        m.store(p.n, to, kept, p.seq.t0);
        return;
    }
    // (units and tables start at different clusters: workgroups 8 apart share an L2 slice, and the same cluster's of all units would meet
    // there.  All 8192 rows in one cluster, 8 / 64 units: 639 / 2412 us unturned, 345 / 541 turned)
    const unsigned turned = (unsigned)(keys ? group - per_table + 4 : group) + (unsigned)u;
    const int f = p.f0 + (int)wrapped(turned, (unsigned)per_table) * 4 + wave;
    const int32_t* start = p.start + u * p.start_stride;
    // (all four clusters' places by every wave: only a workgroup with a long one has anything to say to its other waves)
    int at[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) at[i] = start[min(f - wave + i, p.f1)];
    int s0 = at[0], s1 = at[1];
    bool with_long = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        with_long |= at[i + 1] - at[i] > p.long_cluster;
        if (wave == i) {
            s0 = at[i];
            s1 = at[i + 1];
        }
    }
    const int n = s1 - s0;
    const bool is_long = n > p.long_cluster;
    with_long &= !p.all_by_place;
    if (with_long) {
        if (threadIdx.x < 4) ticket[threadIdx.x] = 0;
        __syncthreads();
    }
    if (f < p.f1) {
        const uint32_t* Xd = reinterpret_cast<const uint32_t*>(X);
        RowSum a;
        if (is_long) {
            a = sum_of_rows<false, 0>(Xd, list, s0, s1, [](int, int, int, uint32_t) {});
        } else {
            uint32_t* to_d = reinterpret_cast<uint32_t*>(to);
            uint32_t* kept_d = reinterpret_cast<uint32_t*>(kept);
            a = sum_of_rows<false, 4>(Xd, list, s0, s1, [&](int at, int q, int row, uint32_t w) {
                store_once(to_d + (long long)at * 64 + (q * 64 + lane), w);
                if (kept && row >= p.seq.t0) store_once(kept_d + (long long)(row - p.seq.t0) * 64 + lane, w);
            });
        }
        const long long table = (long long)u * p.tab_rows + f;
        uint32_t* mean = reinterpret_cast<uint32_t*>(keys ? p.key_means : p.value_means) + table * 64 + lane;
        if (n > 0) *mean = mean_dword(a, n);
        else if (!keys || !p.key_keeps) *mean = 0u;
        if (!keys && lane == 0) p.counts[table] = n;
        double* sums = keys ? p.key_sums : p.value_sums;
        if (sums) {
            double2* to_sums = reinterpret_cast<double2*>(sums + ((long long)u * p.sum_unit_rows + f) * kHeadDim) + lane;
            const double2 both = make_double2(a.a0, a.a1);
            if constexpr (kSumsOnce) store_once(reinterpret_cast<uint4*>(to_sums), __builtin_bit_cast(uint4, both));
            else *to_sums = both;
        }
    }
    if (!with_long) return;
#pragma unroll 1
    for (int w = 0; w < 4; ++w) {
        const int from = start[min(f - wave + w, p.f1)], end = start[min(f - wave + w + 1, p.f1)];
        if (end - from <= p.long_cluster) continue;
        // (a piece's rows are asked for in front of the stores of the one before: loads behind stores would wait for those)
        constexpr int kPiece = 16;
        const int pieces = (end - from + kPiece - 1) / kPiece;
        auto next = [&] {
            int t = 0;
            if (lane == 0) t = atomicAdd(&ticket[w], 1);
            return __builtin_amdgcn_readfirstlane(t);
        };
        auto members = [&](RowMove<kPiece>& m, int t) { m.ask_members(list, from + min(t, pieces - 1) * kPiece, end); };
        if (pieces == 0) continue;
        int t0 = next(), t1 = next();
        if (t0 >= pieces) continue;
        RowMove<kPiece> m0, m1;
        members(m0, t0);
        members(m1, t1);
        m0.ask_rows(X);
        while (true) {
            const int t2 = next();
            RowMove<kPiece> m2;
            members(m2, t2);
            if (t1 < pieces) m1.ask_rows(X);
            m0.store(end, to, kept, p.seq.t0);
            if (t1 >= pieces) break;
            m0 = m1;
            m1.place = m2.place;
            m1.mine = m2.mine;
            t1 = t2;
        }
    }
}

// Stored tables of the coarse clusters [c0, c1), keys (z = 0) and values, from those of their fine clusters (Sec. 3.4: a coarse
// centroid is the mean of all rows below it): one wave per coarse cluster adds its children's fp64 member
// sums in ascending fine id, starting from zero, divides by the children's member count and rounds once
// to bf16.  The key sum of fine cluster f is row (key_map ? key_map[f - f0] : f) of sumK (sums taken before a
// renumbering sit at the old ids).  Empty cluster: `key_fallback` row if given (else zeros).  Lane l owns
// dims 2l and 2l+1, as in cluster_mean_kernel.  Bound by its trips to memory in a row: with every child's place asked for in
// front of its sum, one child after the other, 32 units of 256 fine clusters under 16 coarse ones took 14.3 us, now 6.9.
__global__ __launch_bounds__(256) void coarse_from_children_kernel(const CoarseTables p)
{
    const int u = blockIdx.y;
    const int c = p.c0 + blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= p.c1) return;
    const bool keys = blockIdx.z == 0;
    const int32_t* map = keys ? p.key_map : nullptr;
    const uint16_t* fallback = keys ? p.key_fallback : nullptr;
    const int f_begin = __builtin_amdgcn_readfirstlane(p.cstart[u * p.cstart_stride + c]);
    const int f_end = __builtin_amdgcn_readfirstlane(p.cstart[u * p.cstart_stride + c + 1]);
    const double2* Su = reinterpret_cast<const double2*>((keys ? p.sumK : p.sumV) + (long long)u * p.fcap * kHeadDim);
    int32_t* counts = p.counts + u * p.tab_rows;
    double a0 = 0.0, a1 = 0.0;
    long long n = 0;
    for (int base = f_begin; base < f_end; base += 64) {     // 64 children's sum rows and counts in one trip, a lane each,
        const int here = min(f_end - base, 64), f = base + min(lane, here - 1);
        const int row = map ? map[u * (long long)p.fcap + (f - p.f0)] : f;
        if (lane < here) n += counts[f];
        for (int q0 = 0; q0 < here; q0 += 8) {               // then eight sums in flight, added in order
            double2 w[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                w[q] = Su[(long long)__builtin_amdgcn_readlane(row, min(q0 + q, here - 1)) * 64 + lane];
            asm volatile("" ::"v"(w[6].x), "v"(w[7].x));      // (the last of them, too, before the first is waited for)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q0 + q < here) {
                    a0 += w[q].x;
                    a1 += w[q].y;
                }
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off, 64);
    uint32_t outw;
    if (n > 0) {
        const double inv = (double)n;
        outw = (uint32_t)f64_to_bf16_rne(a0 / inv) | ((uint32_t)f64_to_bf16_rne(a1 / inv) << 16);
    } else if (fallback) {
        outw = reinterpret_cast<const uint32_t*>(fallback + ((long long)u * p.tab_rows + p.fcap + c) * kHeadDim)[lane];
    } else {
        outw = 0u;
    }
    reinterpret_cast<uint32_t*>((keys ? p.Kc : p.Vc) + ((long long)u * p.tab_rows + p.fcap + c) * kHeadDim)[lane] = outw;
    if (!keys && lane == 0) counts[p.fcap + c] = (int32_t)n;
}

// Stored-order tables from member lists built on local point indices, for the fine range [f0, f1) and n_pts points:
// fstart[u][f] = pt0 + start[u][f] for f in [f0, f1];  perm[u][pt0 + p] = pt0 + list[u][p] and fot[u][pt0 + p] = ids[u][p] for
// p < n_pts;  two levels, the coarse ids of the range in [c0, c1) and non-decreasing: cstart[u][c] = first fine id whose coarse
// id is >= c, for c in [c0, c1], cstart[c1] = f1.
__global__ void stored_order_kernel(const StoredOrder p)
{
    const int u = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < p.n_pts) {
        p.perm[u * p.ncap + p.pt0 + i] = p.pt0 + p.list[u * p.ncap + i];
        if (p.ids) p.fot[u * p.ncap + p.pt0 + i] = p.ids[u * p.ids_stride + i];
    }
    if (i > p.f1 - p.f0) return;
    const int f = p.f0 + i;
    p.fstart[u * (long long)(p.fcap + 1) + f] = p.pt0 + p.start[u * p.start_stride + f];
    if (!p.cof) return;
    const int32_t* cof = p.cof + u * (long long)p.fcap;
    const int cur = f < p.f1 ? cof[f] : p.c1, prev = f > p.f0 ? cof[f - 1] : p.c0 - 1;
    for (int c = prev + 1; c <= cur; ++c) p.cstart[u * (long long)(p.ccap + 1) + c] = f;
}

// Rows of several arrays moved in one launch: see CopyBatch.  grid = (pieces of a row, rows, parts)
template <typename T>
__device__ __forceinline__ void copy_row(const CopyBatch::Part& p, unsigned row)
{
    const T* src = reinterpret_cast<const T*>(static_cast<const char*>(p.src) + row * p.spitch);
    T* dst = reinterpret_cast<T*>(static_cast<char*>(p.dst) + row * p.dpitch);
    const unsigned long long n = p.width / sizeof(T);
    for (unsigned long long i = blockIdx.x * (unsigned long long)blockDim.x + threadIdx.x; i < n; i += (unsigned long long)gridDim.x * blockDim.x) dst[i] = src[i];
}
__global__ __launch_bounds__(256) void copy_batch_kernel(const CopyBatch b)
{
    const CopyBatch::Part& p = b.part[blockIdx.z];
    if (p.unit == 16) copy_row<uint4>(p, blockIdx.y);
    else if (p.unit == 4) copy_row<uint32_t>(p, blockIdx.y);
    else copy_row<uint8_t>(p, blockIdx.y);
}

// Dense per-cluster views of the last decode call's selection, from the per-candidate arrays:
// sel[u][id] = flag of the candidate with that id (0 if it was no candidate), r[u][id] = its rank
// key (NaN if it was no candidate).  One workgroup per unit.
__global__ __launch_bounds__(256) void scatter_selection_kernel(const int32_t* __restrict__ cand,
                                                                long long cand_stride,
                                                                const int32_t* __restrict__ n_cand_dev,
                                                                int n_cand_fixed, const uint8_t* __restrict__ flag,
                                                                const unsigned long long* __restrict__ keys,
                                                                const int32_t* __restrict__ key_mode, int level, int G,
                                                                long long pos_stride, int n_ids,
                                                                uint8_t* __restrict__ sel_out, double* __restrict__ r_out)
{
    const int u = blockIdx.x;
    const int n = n_cand_dev ? n_cand_dev[u] : n_cand_fixed;
    const double nan = __longlong_as_double(0x7ff8000000000000ll);
    const int mode = key_mode[2 * u + level];
    const double logG = log((double)G);
    for (int i = threadIdx.x; i < n_ids; i += 256) {
        if (sel_out) sel_out[(long long)u * n_ids + i] = 0;
        if (r_out) r_out[(long long)u * n_ids + i] = nan;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += 256) {
        const int id = cand ? cand[u * cand_stride + i] : i;
        if (sel_out) sel_out[(long long)u * n_ids + id] = flag[u * pos_stride + i];
        if (r_out) {
            const unsigned long long key = keys[u * pos_stride + i];
            double r = nan;
            if (key != ~0ull) {
                if (mode == 1) {
                    r = log(__longlong_as_double((long long)~key)) - logG;
                } else {    // undo the order-preserving map of the rank key
                    unsigned long long b = ~key;
                    b = (b >> 63) ? (b & 0x7fffffffffffffffull) : ~b;
                    r = __longlong_as_double((long long)b);
                }
            }
            r_out[(long long)u * n_ids + id] = r;
        }
    }
}

__global__ __launch_bounds__(256) void fill_kernel(int32_t* __restrict__ dst, int n, int32_t value)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = value;
}

}  // namespace

hipError_t launch_fill(int32_t* dst, int n, int32_t value, hipStream_t s)
{
    hipLaunchKernelGGL(fill_kernel, dim3((n + 255) / 256), dim3(256), 0, s, dst, n, value);
    return hipGetLastError();
}

hipError_t launch_scatter_selection(const int32_t* cand, long long cand_stride, const int32_t* n_cand_dev,
                                    int n_cand_fixed, const uint8_t* flag, const unsigned long long* keys,
                                    const int32_t* key_mode, int level, int G, long long pos_stride, int n_ids, int U,
                                    uint8_t* sel_out, double* r_out, hipStream_t s)
{
    if (n_ids <= 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_selection_kernel, dim3(U), dim3(256), 0, s, cand, cand_stride, n_cand_dev,
                       n_cand_fixed, flag, keys, key_mode, level, G, pos_stride, n_ids, sel_out, r_out);
    return hipGetLastError();
}

// ---- host launchers ----------------------------------------------------------------------------
hipError_t launch_block_lists(const int32_t* ids, long long ids_stride, const int32_t* blocks_dev, int nb,
                              int max_k_per_block, int p_first, int U, int32_t* start, long long start_stride,
                              int32_t* list, long long list_stride, hipStream_t s)
{
    if (nb <= 0 || max_k_per_block <= 0) return hipSuccess;
    constexpr int kLdsInts = 16384;            // 64 KiB
    if (2 * max_k_per_block > kLdsInts) return hipErrorInvalidValue;
    int waves = kLdsInts / max_k_per_block - 1;
    if (waves > kListWaves) waves = kListWaves;
    const size_t smem = (size_t)(waves + 1) * max_k_per_block * sizeof(int32_t);
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&block_lists_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsInts * 4);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL(block_lists_kernel, dim3(nb, U), dim3(1024), smem, s, ids, ids_stride, blocks_dev, p_first,
                       waves, start, start_stride, list, list_stride);
    return hipGetLastError();
}

// A cluster's wave that also stores its rows is the longer chain, and moves a row's bytes once less: it pays where the waves fill the chip.
// Us, rows stored by place / by clusters, tables of keys and values given their clustering: 1 unit of 256 clusters 34.8 / 36.7, 2 of 256
// 37.1 / 38.1, 4 of 256 42.3 / 41.9, 8 of 256 56.2 / 52.3, 64 of 256 217 / 185; builds of five iterations, values only: 1 x 46 148.4 / 154.4,
// 8 x 128 284 / 287, 16 x 256 460 / 464, 8 x 1024 613.9 / 610.7, 64 x 256 817 / 807.
constexpr int kFewClustersOfTwo = 768, kFewClustersOfOne = 6144;      // of all units
// Clusters of all units whose sums (a kilobyte a table) do not stay in the 256 MiB last-level cache until the coarse tables are added up from
// them: they are stored past it.  Us, through it / past it, two levels, both tables: 64 units of 2048 clusters 384 / 392, 16 of 8000 838 / 850, 64 of
// 2730 493 / 481, 64 of 4096 678 / 660, 256 of 700 475 / 468, 32 of 8192 993 / 972, 128 of 3000 864 / 833.
constexpr long long kCachedSums = 150000;
hipError_t launch_stored_rows(StoredRows p, int U, hipStream_t s)
{
    if (p.n <= 0 || p.f1 <= p.f0) return hipSuccess;
    p.long_cluster = std::max(128, 4 * (p.n / (p.f1 - p.f0)));
    const int per_table = (p.f1 - p.f0 + 3) / 4, places = (p.n + 4 * kMoveRows - 1) / (4 * kMoveRows);
    p.all_by_place = (long long)U * (p.f1 - p.f0) <= (p.key_means ? kFewClustersOfTwo : kFewClustersOfOne);
    if (p.all_by_place) p.long_cluster = -1;
    const int groups = per_table * (p.key_means ? 2 : 1) + places * (p.all_by_place ? 2 : p.key_means ? 0 : 1);
    const bool past = (p.key_means ? p.key_sums : p.value_sums) && (long long)U * (p.f1 - p.f0) * (p.key_means ? 2 : 1) > 2 * kCachedSums;
    if (past) hipLaunchKernelGGL(stored_rows_kernel<true>, dim3(groups, U), dim3(256), 0, s, p);
    else hipLaunchKernelGGL(stored_rows_kernel<false>, dim3(groups, U), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_gather_quantize_rows(const void* srcK, const void* srcV, long long src_unit_rows, const int32_t* list,
                                       long long list_stride, const int32_t* ids, long long ids_stride,
                                       const uint16_t* Kc, long long kc_unit_rows, int n, int U, void* dstK, void* dstV,
                                       float* scales, long long dst_unit_rows, int dst_row0, const SequenceCopy& seq,
                                       int32_t* unusual, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const long long threads = (long long)n * 16;
    hipLaunchKernelGGL(gather_quantize_rows_kernel, dim3((unsigned)((threads + 255) / 256), U), dim3(256), 0, s,
                       (const uint4*)srcK, (const uint4*)srcV, src_unit_rows, list, list_stride, ids, ids_stride,
                       (const uint4*)Kc, kc_unit_rows, n, (uint2*)dstK, (uint2*)dstV, (float2*)scales, dst_unit_rows,
                       dst_row0, seq, unusual);
    return hipGetLastError();
}

hipError_t launch_cluster_means(const uint16_t* X, long long x_unit_rows, const int32_t* list, long long list_stride,
                                const int32_t* start, long long start_stride, int k0, int k, int U,
                                uint16_t* mean_out, long long out_unit_rows, int out_row0, const uint16_t* fallback,
                                long long fb_unit_rows, int32_t* count_out, long long count_stride, int count_off,
                                double* sum_out, long long sum_unit_rows, uint32_t* range_out, uint32_t* changed_out, hipStream_t s)
{
    if (k <= k0) return hipSuccess;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((k - k0 + 3) / 4, U), dim3(256), 0, s, X, x_unit_rows, list, list_stride, start,
                           start_stride, k0, k, mean_out, out_unit_rows, out_row0, fallback, fb_unit_rows, count_out,
                           count_stride, count_off, sum_out, sum_unit_rows, range_out, changed_out);
        return hipGetLastError();
    };
    return range_out ? go(cluster_mean_kernel<true>) : go(cluster_mean_kernel<false>);
}

hipError_t launch_coarse_from_children(const CoarseTables& p, int U, hipStream_t s)
{
    if (p.c1 <= p.c0) return hipSuccess;
    hipLaunchKernelGGL(coarse_from_children_kernel, dim3((p.c1 - p.c0 + 3) / 4, U, 2), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_stored_order(const StoredOrder& p, int U, hipStream_t s)
{
    const int n = p.n_pts > p.f1 - p.f0 + 1 ? p.n_pts : p.f1 - p.f0 + 1;
    hipLaunchKernelGGL(stored_order_kernel, dim3((n + 255) / 256, U), dim3(256), 0, s, p);
    return hipGetLastError();
}

void CopyBatch::add(void* dst, size_t dpitch, const void* src, size_t spitch, size_t width)
{
    if (width == 0) return;
    const size_t all = (uintptr_t)dst | dpitch | (uintptr_t)src | spitch | width;
    part[n++] = Part{src, dst, (long long)spitch, (long long)dpitch, width, all % 16 == 0 ? 16u : all % 4 == 0 ? 4u : 1u};
}

hipError_t CopyBatch::launch(int rows, hipStream_t s)
{
    if (n == 0 || rows == 0) return hipSuccess;
    unsigned long long most = 1;
    for (int i = 0; i < n; ++i) most = std::max<unsigned long long>(most, part[i].width / part[i].unit);
    // (up to four pieces a thread: enough workgroups to fill the chip in any case that takes longer than a launch)
    const unsigned gx = (unsigned)std::min<unsigned long long>((most + 1023) / 1024, 4096);
    hipLaunchKernelGGL(copy_batch_kernel, dim3(gx, rows, n), dim3(256), 0, s, *this);
    n = 0;
    return hipGetLastError();
}

}  // namespace mp
