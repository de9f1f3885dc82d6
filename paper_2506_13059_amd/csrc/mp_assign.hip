// Nearest-centroid assignment of k-means on the keys (Sec. 3.1: assignment step of Lloyd's iterations;
// Sec. 3.3: run inside each block of the sequence, and as the one-shot assignment of appended tokens).
//
// The result is defined in fp64: a[t] = argmin_j sum_i (x_t[i] - c_j[i])^2 with the sum taken in
// index order and the lowest j among equal distances.  Points and centroids are bf16 values, so the
// bulk of the work is a bf16 contraction and runs on the matrix cores; fp64 is only spent where it
// can change the answer:
//
//   1. assign_mfma_kernel: s[t,j] = x_t.c_j - |c_j|^2/2 (argmax = nearest centroid) with
//      v_mfma_f32_32x32x16_bf16, fp32 accumulation.  The offset -|c_j|^2/2 is part of the
//      contraction: split exactly into three bf16 values, it sits in three extra slots of the
//      reduction dimension against ones on the point side, so the scores leave the matrix cores
//      complete.  Per point the kernel keeps the best and the second best score.  A point whose two
//      best scores are further apart than the margin of mp_margin.h (2^-14 of max(|x|^2,
//      max_j |c_j|^2), 1.1 times what the two can be off together) has a unique nearest centroid in
//      exact arithmetic too (and by far more than fp64 rounding), which is the fp64 answer.
//   2. Every other point (near-equal or equal distances) goes onto a per-block list and
//      assign_recheck_kernel decides it exactly as defined above: it collects the centroids whose
//      score is within the same margin of the best one and evaluates their distances in fp64
//      without fused multiply-adds.  (Kernels that hold a block's centroids do this themselves.)
#include <algorithm>
#include <type_traits>

#include "mp_device.h"
#include "mp_internal.h"
#include "mp_margin.h"
#include "mp_plan.h"

namespace mp {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kTile = 32;                 // centroids per tile = rows of the MFMA A operand
constexpr int kRowBytes = 256 + 16;       // LDS row of one centroid: 128 dims, then -|c|^2/2 as three bf16 and five zeros
constexpr uint32_t kTiledSlotMask = (1u << kTiledSlotBits) - 1u;
constexpr float kNoCentroid = -3.0e38f;          // score of a padded row (finite: index bits are packed into scores)

// Scores of 32 centroids (one LDS tile: rows of kRowBytes, -|c|^2/2 in three bf16 pieces behind the
// 128 dims) against this wave's 2 x 32 points, folded into the running best / second best of every
// point.  Accumulator rows of a lane: m(i) = 8 (i / 4) + 4 half + i % 4.  The slot i of a score
// inside the tile rides in its four lowest mantissa bits (a change of at most 2^-19 of its
// magnitude), so that a pair of scores costs one max3, one med3 and one max; the tile of the best
// score is noted per tile.
__device__ __forceinline__ void fold_scores(const f32x16_t (&acc)[2], int j0, float (&best)[2], float (&second)[2],
                                            int (&btile)[2])
{
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float before = best[c];
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float va = __uint_as_float((__float_as_uint(acc[c][i]) & ~kTiledSlotMask) | (uint32_t)i);
            const float vb = __uint_as_float((__float_as_uint(acc[c][i + 1]) & ~kTiledSlotMask) | (uint32_t)(i + 1));
            second[c] = fmaxf(second[c], __builtin_amdgcn_fmed3f(best[c], va, vb));
            best[c] = fmaxf(fmaxf(va, vb), best[c]);
        }
        btile[c] = best[c] != before ? j0 : btile[c];
    }
}

__device__ __forceinline__ void tile_scores(const unsigned char* tile, int col, int half, const bf16x8_t (&xb)[2][8],
                                            bf16x8_t ones, bf16x8_t ones_too, int j0, float (&best)[2],
                                            float (&second)[2], int (&btile)[2])
{
    f32x16_t acc[2];
    {
        const f32x16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(tile + col * kRowBytes + 256);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, ones, zero, 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, ones_too, zero, 0, 0, 0);
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(tile + col * kRowBytes + 32 * ks + 16 * half);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xb[0][ks], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xb[1][ks], acc[1], 0, 0, 0);
    }
    fold_scores(acc, j0, best, second, btile);
}

// One 16-byte piece of a centroid row goes to its place in an LDS tile; the 16 lanes that hold a
// row add up |c|^2 (exact products, a dozen fp32 roundings: at most 2^-20 of its value, far below
// the bound on a score), and the lane with the first piece writes -|c|^2/2 behind the row, split
// exactly into three bf16 values (24 significant bits in three pieces of 8).  Returns |c|^2.
__device__ __forceinline__ float deposit_piece(unsigned char* tile_row, int seg, uint4 w, bool exists)
{
    *reinterpret_cast<uint4*>(tile_row + seg * 16) = w;
    float s = dot2_bf16(w.x, w.x, 0.f);
    s = dot2_bf16(w.y, w.y, s);
    s = dot2_bf16(w.z, w.z, s);
    s = dot2_bf16(w.w, w.w, s);
    s = sum8(s);
    s += dpp_f32<kDppMirror>(s);      // the other 8 lanes of the row of 16
    if (seg == 0) {
        const float v = exists ? -0.5f * s : kNoCentroid;
        const uint32_t hi = __float_as_uint(v) & 0xffff0000u;
        const float r1 = v - __uint_as_float(hi);
        const uint32_t mid = __float_as_uint(r1) & 0xffff0000u;
        const uint32_t lo = __float_as_uint(r1 - __uint_as_float(mid)) & 0xffff0000u;
        *reinterpret_cast<uint4*>(tile_row + 256) = make_uint4((hi >> 16) | mid, lo >> 16, 0u, 0u);
    }
    return s;
}

// The chunks [first, end) of 64 points of a block that has not changed since the last step: the same ids, no marks.
__device__ __forceinline__ bool unchanged(const MoveMarks& mv, int u, int b, int cnt_stride)
{
    return mv.marks && mv.moved_before && mv.moved_before[u * cnt_stride + b] == 0;
}
__device__ __forceinline__ void keep_chunks(const MoveMarks& mv, int u, int b, int x0, int x1, int first, int end, int32_t* assign,
                                            long long assign_stride)
{
    for (int t = x0 + 64 * first + (int)threadIdx.x; t < min(x0 + 64 * end, x1); t += (int)blockDim.x)
        assign[u * assign_stride + t] = mv.old_ids[u * assign_stride + t];
    for (int c = first + (int)threadIdx.x; c < end; c += (int)blockDim.x) mv.marks[u * mv.stride + first_mark(x0, b) + c] = 0;
}

// The two halves of a wave hold the other accumulator rows of the same points: combine them, write
// the stage-1 assignment, and list the point for the exact pass unless its two best scores are
// further apart than the margin.
__device__ __forceinline__ void finish_points(int half, const float (&best)[2], const float (&second)[2],
                                              const int (&btile)[2], const float (&x2)[2], const int (&tpt)[2], int x0,
                                              int x1, float c2max, int32_t* assign_u, int32_t* amb_list_u,
                                              int32_t* amb_cnt_ub, const int32_t* old_u, unsigned long long* mark)
{
    unsigned long long marked = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int slot = (int)(__float_as_uint(best[c]) & kTiledSlotMask);
        const int bj = btile[c] + 8 * (slot >> 2) + 4 * half + (slot & 3);
        const float ob = __shfl_xor(best[c], 32, 64), os = __shfl_xor(second[c], 32, 64);
        const int oj = __shfl_xor(bj, 32, 64);
        const float ox = __shfl_xor(x2[c], 32, 64);
        const float sec = fmaxf(fmaxf(second[c], os), fminf(best[c], ob));
        int j = bj;
        if (ob > best[c] || (ob == best[c] && oj < j)) j = oj;
        const float bst = fmaxf(best[c], ob);
        const float xx = x2[c] + ox;
        const int t = tpt[c];
        bool moved = false;
        if (t < x1 && half == 0) {
            assign_u[t] = j;
            const float margin = near_margin(fmaxf(xx, c2max));
            // (written so that a point without any comparable score also goes to the exact pass)
            const bool near = !(bst - sec > margin);
            if (near) {
                const int pos = atomicAdd(amb_cnt_ub, 1);
                amb_list_u[x0 + pos] = t;
            }
            moved = near || (mark && old_u[t] != j);
        }
        marked |= __ballot(moved) << (32 * c);               // (the lower half has a bit of each of its 32 points)
    }
    if (mark && (threadIdx.x & 63) == 0) *mark = marked;
}

// grid = (ceil(max points per block / 256), nb, U); 256 threads = 4 waves of 64 points (two MFMA
// column tiles that share every centroid fragment).  Centroid tiles are double-buffered in LDS; their
// rows are requested two tiles ahead and wait in registers until the buffer they go to is free.
// blocks: int32 [nb][4] = {first point, end point, first centroid, end centroid}.
// assign[u][t] receives the best centroid of stage 1; amb_list[u][first point + i], i < amb_cnt[u][b],
// the points of block b that stage 2 has to decide.
constexpr int kPtsPerWg = 256;
__global__ __launch_bounds__(256) void assign_mfma_kernel(const uint16_t* __restrict__ X, long long x_unit_rows,
                                                          const int32_t* __restrict__ blocks,
                                                          const uint16_t* __restrict__ C, long long c_unit_rows,
                                                          int32_t* __restrict__ assign, long long assign_stride,
                                                          int32_t* __restrict__ amb_list, long long list_stride,
                                                          int32_t* __restrict__ amb_cnt, int cnt_stride, const MoveMarks mv)
{
    __shared__ __align__(16) unsigned char tile[2][kTile * kRowBytes];
    __shared__ float wave_c2max[4];
    const int u = blockIdx.z, b = blockIdx.y;
    const int x0 = blocks[4 * b + 0], x1 = blocks[4 * b + 1], k0 = blocks[4 * b + 2], k1 = blocks[4 * b + 3];
    const int p0 = x0 + (int)blockIdx.x * kPtsPerWg;
    if (p0 >= x1) return;
    if (mv.marks && blockIdx.x == 0 && threadIdx.x == 0) mv.moved_now[u * cnt_stride + b] = 0;
    if (unchanged(mv, u, b, cnt_stride)) {
        keep_chunks(mv, u, b, x0, x1, (p0 - x0) / 64, min((p0 - x0 + kPtsPerWg) / 64, (x1 - x0 + 63) / 64), assign, assign_stride);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;

    // B operands: this lane's two points, dims [16 ks + 8 half, +8) for ks = 0..7
    bf16x8_t xb[2][8];
    float x2[2];
    int tpt[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        tpt[c] = p0 + wave * 64 + 32 * c + col;
        const int tl = tpt[c] < x1 ? tpt[c] : x0;
        const uint4* xp = reinterpret_cast<const uint4*>(X + ((long long)u * x_unit_rows + tl) * kHeadDim);
        x2[c] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const uint4 w = xp[2 * ks + half];
            xb[c][ks] = __builtin_bit_cast(bf16x8_t, w);
            x2[c] = dot2_bf16(w.x, w.x, x2[c]);      // |x|^2 only scales the margin
            x2[c] = dot2_bf16(w.y, w.y, x2[c]);
            x2[c] = dot2_bf16(w.z, w.z, x2[c]);
            x2[c] = dot2_bf16(w.w, w.w, x2[c]);
        }
    }
    // point side of the three offset slots: ones in the slots of the lower half-wave, zeros elsewhere
    const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, half == 0 ? make_uint4(0x3f803f80u, 0x00003f80u, 0u, 0u)
                                                                  : make_uint4(0u, 0u, 0u, 0u));
    bf16x8_t ones_too = ones;      // a second copy the compiler cannot see through: two multiplications
    asm volatile("" : "+v"(ones_too));   // on the otherwise idle matrix pipe instead of sixteen register moves
    // this thread's share of a centroid tile: two 16-byte pieces, 16 threads per row
    const uint16_t* Cu = C + (long long)u * c_unit_rows * kHeadDim;
    uint4 pre_a[2], pre_b[2];     // rows on their way to LDS: the next tile and the one after it
    float c2max = 0.f;
    auto request = [&](int j0, uint4 (&pre)[2]) {
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const int e = pass * 256 + tid;
            const int row = e >> 4, seg = e & 15;
            // always a load (of the last centroid when the row does not exist; deposit stores zeros for
            // it): the count of loads in flight is then the same on every path, which is what lets
            // the compiler wait for the older request only
            const int j = j0 + row < k1 ? j0 + row : k1 - 1;
            pre[pass] = reinterpret_cast<const uint4*>(Cu + (long long)j * kHeadDim)[seg];
        }
    };
    auto deposit = [&](int j0, int buf, const uint4 (&pre)[2]) {
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const int e = pass * 256 + tid;
            const int row = e >> 4, seg = e & 15;
            const bool exists = j0 + row < k1;
            const uint4 w = exists ? pre[pass] : make_uint4(0, 0, 0, 0);
            c2max = fmaxf(c2max, deposit_piece(tile[buf] + row * kRowBytes, seg, w, exists));   // (absent rows are zeros)
        }
    };
    float best[2] = {-INFINITY, -INFINITY}, second[2] = {-INFINITY, -INFINITY};
    int btile[2] = {k0, k0};
    // Rows are requested two tiles ahead: a tile's multiplications take less time than a load from
    // L2 under the traffic of the other workgroups' point loads.
    request(k0, pre_a);
    request(k0 + kTile, pre_b);
    deposit(k0, 0, pre_a);
    __syncthreads();
    // one tile: `next` holds the rows of the following tile, `after` receives those of the one after it
    auto step = [&](int j0, int buf, uint4 (&after)[2], const uint4 (&next)[2]) {
        const bool more = j0 + kTile < k1;
        request(j0 + 2 * kTile, after);
        __builtin_amdgcn_sched_barrier(0);      // (the compiler would sink the loads below the multiplications)
        tile_scores(tile[buf], col, half, xb, ones, ones_too, j0, best, second, btile);
        if (more) deposit(j0 + kTile, buf ^ 1, next);
        __syncthreads();
    };
    // (two tiles per trip, so that the two register sets swap roles without being copied: a copy
    // would have to wait for the load)
    for (int j0 = k0; j0 < k1; j0 += 2 * kTile) {
        step(j0, 0, pre_a, pre_b);
        if (j0 + kTile < k1) step(j0 + kTile, 1, pre_b, pre_a);
    }
    // largest |c|^2 of the block: every thread saw the rows it deposited
    c2max = wave_max_f32(c2max);
    if (lane == 0) wave_c2max[wave] = c2max;
    __syncthreads();
    c2max = fmaxf(fmaxf(wave_c2max[0], wave_c2max[1]), fmaxf(wave_c2max[2], wave_c2max[3]));
    const int chunk = (p0 - x0) / 64 + wave;
    finish_points(half, best, second, btile, x2, tpt, x0, x1, c2max, assign + u * assign_stride,
                  amb_list + u * list_stride, amb_cnt + u * cnt_stride + b, mv.old_ids + u * assign_stride,
                  mv.marks && 64 * chunk < x1 - x0 ? mv.marks + u * mv.stride + first_mark(x0, b) + chunk : nullptr);
}

// The same stage for blocks of at most 512 centroids and at least 1024 points.  The block's centroids stay in LDS
// (256-byte rows, 16-byte pieces at position piece ^ (row & 15), and -|c|^2/2 apart: it is the accumulators' initial
// value), every wave walks chunks of 64 points held in registers as B operands, no barrier after the centroids are in
// place.  16 x 16 products: a load instruction of the points covers 64 contiguous bytes of 16 rows, and a tile's
// accumulators are few enough for four waves a SIMD, which hide each other's loads, LDS reads and comparisons.
//
// What bounds it: per tile of 16 centroids x 64 points 16 matrix instructions (16 cycles each) and 36 comparison
// instructions (16 to place the slot, 20 for best and second best).  The two overlap across waves -- a loop
// of 4 32x32x16 products and 32 vector instructions takes 299 ns for four waves, 219 and 236 ns apart -- so occupancy and instruction
// count decide: with two waves a SIMD, 32 x 32 products and 79 vector instructions per 2048 scores 1330 us for 16.8 M
// points x 256 centroids; points streamed through LDS and centroids in registers, two waves, 1390; this
// layout with three waves 1352, with four waves 1044 us (38.6 -> 27.3 us for 262144 points); these figures are without
// the near ties, with them a launch takes 1142 to 1183 us and 36.3 us (nearest_exact).  The points alone take 0.65 ms at
// the rate of the dense kernel; clocks fall to about 2.0 GHz under this load.
//
// A lane (g, c) holds rows 4g .. 4g+3 of a tile for column c of four columns groups: point 16 q + c, q < 4.  The slot of a
// score among the sixteen tiles of a half (tile & 15, row & 3) rides in its six lowest mantissa bits, a change of less
// than 2^-17 of its magnitude, which the margin covers (near_margin_of_best).
constexpr int kRowTile = 16;
constexpr int kHalfTiles = 16;                   // tiles whose slots fit the six bits
constexpr int kNearCap = 256;                    // (a multiple of sixteen)
constexpr int kResidentTwiceK = 304;             // 2 x (304 x 260 + 2.6 K) bytes of the compute unit's 160 KiB
constexpr int kCoarseLds = 160 * 1024 - 2048;    // of a compute unit, less what the coarse level's kernel has besides
constexpr int kChangedTwiceK = 288;              // 2 x (288 x 268 + 1.6 K)
constexpr uint32_t kSlotMask = (1u << kResidentSlotBits) - 1u;

typedef const __attribute__((address_space(3))) bf16x8_t lds_frag;
typedef const __attribute__((address_space(3))) f32x4_t lds_four;
// (plain operations, no inline assembly: only the compiler knows how long a matrix result must not be read)
__device__ __forceinline__ float with_slot(float v, uint32_t clear, uint32_t slot)
{
    return __uint_as_float((__float_as_uint(v) & clear) | slot);
}
__device__ __forceinline__ void swap_halves(float& a, float& b)      // a = {a.low, b.low}, b = {a.high, b.high}
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows(float& a, float& b)        // the same with rows 1, 3 of a and 0, 2 of b
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
// Two candidates (best, second, origin bits) of the same point become one; `bit` marks that the second one won.
__device__ __forceinline__ void merge_pair(float& best, float& second, uint32_t& from, float best2, float second2, uint32_t from2,
                                           uint32_t bit)
{
    second = fmaxf(fmaxf(second, second2), fminf(best, best2));
    from = best2 > best ? (from2 | bit) : from;
    best = fmaxf(best, best2);
}

// Where the points are: 16-byte piece i of point t (of the unit, or of the block where its points are in LDS).
struct PointsInMemory {
    const unsigned char* Xu;
    __device__ __forceinline__ uint4 piece(int t, int i) const { return reinterpret_cast<const uint4*>(Xu + (long long)t * 256)[i]; }
};
struct PointsInLds {      // (256-byte rows swizzled as the centroids')
    const unsigned char* rows;
    __device__ __forceinline__ uint4 piece(int t, int i) const { return *reinterpret_cast<const uint4*>(rows + t * 256 + ((i ^ t) & 15) * 16); }
};

// The nearest of the centroids in LDS (rows at lds0, -|c|^2/2 at ci0) for the 64 points first, first + 1, ...
// (clamped to `last`): lane = point.  `near`: its two best scores are closer than the margin.
struct Nearest {
    int j;
    bool near;
    float best, second;      // the best scores (their lowest bits carry the slot)
    float m;                 // what margins grow with: the largest of |x|^2 and c2max
};
template <typename Points>
__device__ __forceinline__ Nearest nearest_of_chunk(const Points& X, int first, int last, uint32_t lds0, uint32_t ci0,
                                                    int ntiles, float c2max)
{
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    uint32_t clear = ~kSlotMask;
    asm volatile("" : "+v"(clear));              // (a register: the instruction takes one scalar operand, the slot)
    bf16x8_t x[4][4];                        // points 16 q + c, dims [32 ks + 8 g, +8)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int t = min(first + 16 * q + c, last);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) x[q][ks] = __builtin_bit_cast(bf16x8_t, X.piece(t, 4 * ks + g));
    }
    float best[4], second[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) best[q] = second[q] = -INFINITY;
    // |x|^2 only scales the margin; lane = point after the reduction
    float n2[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        n2[q] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const uint4 w = __builtin_bit_cast(uint4, x[q][ks]);
            n2[q] = dot2_bf16(w.x, w.x, n2[q]);
            n2[q] = dot2_bf16(w.y, w.y, n2[q]);
            n2[q] = dot2_bf16(w.z, w.z, n2[q]);
            n2[q] = dot2_bf16(w.w, w.w, n2[q]);
        }
    }
    auto one_tile = [&](const uint32_t (&fr)[4], uint32_t ci_at, auto step, uint32_t slot) {
        constexpr int kStep = decltype(step)::value;
        bf16x8_t f[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) f[ks] = *reinterpret_cast<lds_frag*>((uintptr_t)(fr[ks] + kStep * kRowTile * 256));
        const f32x4_t ci = *reinterpret_cast<lds_four*>((uintptr_t)(ci_at + kStep * kRowTile * 4));
        f32x4_t acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[0], x[q][0], ci, 0, 0, 0);
#pragma unroll
        for (int ks = 1; ks < 4; ++ks)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[ks], x[q][ks], acc[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = with_slot(acc[q][i], clear, slot + 4u * kStep + i);
            // best and second best of the running pair and four scores: five instructions
            const float m0 = __builtin_amdgcn_fmed3f(best[q], v[0], v[1]);
            best[q] = fmaxf(fmaxf(v[0], v[1]), best[q]);
            const float m1 = __builtin_amdgcn_fmed3f(best[q], v[2], v[3]);
            best[q] = fmaxf(fmaxf(v[2], v[3]), best[q]);
            second[q] = fmaxf(fmaxf(m0, m1), second[q]);
        }
    };
    auto tiles = [&](int ta, int tb) {
        uint32_t fr[4], ci_at = ci0 + (uint32_t)((ta * kRowTile + 4 * g) * 4);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            fr[ks] = lds0 + (uint32_t)(ta * kRowTile * 256 + c * 256 + ((g ^ c) & 3) * 16 + ((64 * ks) ^ ((c >> 2) * 64)));
        uint32_t slot = 0;
        int t = ta;
#pragma unroll 1
        for (; t + 4 <= tb; t += 4) {
            one_tile(fr, ci_at, std::integral_constant<int, 0>{}, slot);
            one_tile(fr, ci_at, std::integral_constant<int, 1>{}, slot);
            one_tile(fr, ci_at, std::integral_constant<int, 2>{}, slot);
            one_tile(fr, ci_at, std::integral_constant<int, 3>{}, slot);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) fr[ks] += 4 * kRowTile * 256;
            ci_at += 4 * kRowTile * 4;
            slot += 16u;
        }
#pragma unroll 1
        for (; t < tb; ++t) {
            one_tile(fr, ci_at, std::integral_constant<int, 0>{}, slot);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) fr[ks] += kRowTile * 256;
            ci_at += kRowTile * 4;
            slot += 4u;
        }
    };
    tiles(0, min(ntiles, kHalfTiles));
    uint32_t from[4] = {0u, 0u, 0u, 0u};
    if (ntiles > kHalfTiles) {
        float first_half[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) first_half[q] = best[q];
        tiles(kHalfTiles, ntiles);
#pragma unroll
        for (int q = 0; q < 4; ++q) from[q] = best[q] != first_half[q] ? 4u : 0u;
    }
    // lane (g, c) ends up with point 16 g + c = lane: halves first (points q and q + 2), then rows
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        float fl = __uint_as_float(from[q]), fh = __uint_as_float(from[q + 2]);
        swap_halves(best[q], best[q + 2]);
        swap_halves(second[q], second[q + 2]);
        swap_halves(n2[q], n2[q + 2]);
        swap_halves(fl, fh);
        from[q] = __float_as_uint(fl);
        merge_pair(best[q], second[q], from[q], best[q + 2], second[q + 2], __float_as_uint(fh), 2u);
        n2[q] += n2[q + 2];
    }
    {
        float fl = __uint_as_float(from[0]), fh = __uint_as_float(from[1]);
        swap_rows(best[0], best[1]);
        swap_rows(second[0], second[1]);
        swap_rows(n2[0], n2[1]);
        swap_rows(fl, fh);
        from[0] = __float_as_uint(fl);
        merge_pair(best[0], second[0], from[0], best[1], second[1], __float_as_uint(fh), 1u);
        n2[0] += n2[1];
    }
    const uint32_t slot = __float_as_uint(best[0]) & kSlotMask;
    const int tile = (int)(slot >> 2) + (int)(from[0] >> 2) * kHalfTiles, row_g = (int)(from[0] & 3u);
    const float m = fmaxf(n2[0], c2max), margin = near_margin_of_best(m, best[0]);
    // (written so that a point without any comparable score also goes to the exact pass)
    return Nearest{tile * kRowTile + 4 * row_g + (int)(slot & 3u), !(best[0] - second[0] > margin), best[0], second[0], m};
}

// One 16-byte piece of a centroid row (16 lanes per row) to its place in LDS; the lane with the first piece writes
// -|c|^2/2.  Returns |c|^2.
__device__ __forceinline__ float place_centroid(unsigned char* rows_lds, float* c_init, int row, int seg, uint4 w, bool exists)
{
    *reinterpret_cast<uint4*>(rows_lds + row * 256 + ((seg ^ row) & 15) * 16) = w;
    float s = dot2_bf16(w.x, w.x, 0.f);
    s = dot2_bf16(w.y, w.y, s);
    s = dot2_bf16(w.z, w.z, s);
    s = dot2_bf16(w.w, w.w, s);
    s = sum8(s);
    s += dpp_f32<kDppMirror>(s);         // the other 8 lanes of the row of 16
    if (seg == 0) c_init[row] = exists ? -0.5f * s : kNoCentroid;
    return s;
}

// |x - c|^2 in fp64 as in exact_distance, the centroid in LDS
template <typename Points>
__device__ __forceinline__ double exact_distance_lds(const Points& X, int t, const unsigned char* rows_lds, int j)
{
    double s = 0.0;
#pragma unroll 4
    for (int i = 0; i < 16; ++i) {
        const uint4 xw = X.piece(t, i), cw = *reinterpret_cast<const uint4*>(rows_lds + j * 256 + ((i ^ j) & 15) * 16);
        const uint32_t c4[4] = {cw.x, cw.y, cw.z, cw.w}, x4[4] = {xw.x, xw.y, xw.z, xw.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double d0 = __dsub_rn((double)bf16lo_to_f32(x4[e]), (double)bf16lo_to_f32(c4[e]));
            const double d1 = __dsub_rn((double)bf16hi_to_f32(x4[e]), (double)bf16hi_to_f32(c4[e]));
            s = __dadd_rn(s, __dmul_rn(d0, d0));
            s = __dadd_rn(s, __dmul_rn(d1, d1));
        }
    }
    return s;
}

// (counted anew: as the thread's index it would be kept in a register through the loop before, which has none left)
__device__ __forceinline__ int lane_id()
{
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// The near ties decided exactly, sixteen points a wave: lane (g, c) has point t of column c (the same in its four lanes)
// and rows 4 g + i of every tile.  Scores again, their maximum, and every centroid within the margin of it is a
// candidate, a bit in its lane's mask: the nearest centroid in exact arithmetic, and everything tied with it, is among
// them.  Then the candidates' distances as defined, one of every lane at a time; smallest distance, equal distances ->
// lowest index.  Returns it in all four lanes.
// A launch of its own fetched the 64 KiB of a block's centroids for every point: 14.6 us for 32 blocks of 8192 points,
// 140 us for 2048.  Here it adds 9 us to the first's assignment (the longest chain: four tiles' products, compared, four
// more, then two or three distances of 2 us) and about 100 to 140 to the second's (1044 us without near ties, 1142 to 1183
// with them).
// known: `best` is what nearest_of_chunk found, at most 2^-17 of its size off, and need not be looked for again.
// id_of: the cluster whose centroid stands at a place of the rows.
template <typename Points, typename IdOf>
__device__ __forceinline__ int nearest_exact(const Points& X, int t, const unsigned char* rows_lds, uint32_t lds0, uint32_t ci0,
                                             int k, float c2max, bool known, float best, IdOf id_of)
{
    const int lane = lane_id(), c = lane & 15, g = lane >> 4;
    const int ntiles = (k + kRowTile - 1) / kRowTile;
    bf16x8_t x[4];
    float n2 = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const uint4 w = X.piece(t, 4 * ks + g);
        x[ks] = __builtin_bit_cast(bf16x8_t, w);
        n2 = dot2_bf16(w.x, w.x, n2);
        n2 = dot2_bf16(w.y, w.y, n2);
        n2 = dot2_bf16(w.z, w.z, n2);
        n2 = dot2_bf16(w.w, w.w, n2);
    }
    n2 += __shfl_xor(n2, 16, 64);
    n2 += __shfl_xor(n2, 32, 64);
    const uint32_t at = lds0 + (uint32_t)(c * 256 + ((g ^ c) & 3) * 16), turn = (uint32_t)((c >> 2) * 64);
    auto scores = [&](int tile) {
        f32x4_t acc = *reinterpret_cast<lds_four*>((uintptr_t)(ci0 + (uint32_t)((tile * kRowTile + 4 * g) * 4)));
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const bf16x8_t f = *reinterpret_cast<lds_frag*>((uintptr_t)(at + (uint32_t)(tile * kRowTile * 256) + ((uint32_t)(64 * ks) ^ turn)));
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, x[ks], acc, 0, 0, 0);
        }
        return acc;
    };
    if (!known) {
        best = -INFINITY;
        for (int tile = 0; tile < ntiles; tile += 4) {
            f32x4_t s[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] = scores(min(tile + r, ntiles - 1));
#pragma unroll
            for (int r = 0; r < 4; ++r) best = fmaxf(best, fmaxf(fmaxf(s[r][0], s[r][1]), fmaxf(s[r][2], s[r][3])));
        }
        best = fmaxf(best, __shfl_xor(best, 16, 64));
        best = fmaxf(best, __shfl_xor(best, 32, 64));
    }
    const float thr = best - near_margin(fmaxf(n2, c2max)) - fabsf(best) * (1.0f / 65536.0f);
    double bd = INFINITY;
    int bj = 0;
    for (int t0 = 0; t0 < ntiles; t0 += 16) {
        unsigned long long mask = 0;
        const int t1 = min(t0 + 16, ntiles);
        for (int tile = t0; tile < t1; tile += 4) {
            f32x4_t s[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] = scores(min(tile + r, ntiles - 1));
            uint32_t bits = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) bits |= (!(s[r][i] < thr) && (tile + r) * kRowTile + 4 * g + i < k) ? 1u << (4 * r + i) : 0u;
            mask |= (unsigned long long)bits << (4 * (tile - t0));
        }
        while (__any(mask != 0)) {
            if (mask != 0) {
                const int e = __ffsll(mask) - 1;
                mask &= mask - 1;
                const int j = (t0 + (e >> 2)) * kRowTile + 4 * g + (e & 3);
                const double d = exact_distance_lds(X, t, rows_lds, j);
                const int id = id_of(j);
                if (d < bd || (d == bd && id < bj)) { bd = d; bj = id; }
            }
        }
    }
#pragma unroll
    for (int off = 32; off >= 16; off >>= 1) {
        const double od = __shfl_xor(bd, off, 64);
        const int oj = __shfl_xor(bj, off, 64);
        if (od < bd || (od == bd && oj < bj)) { bd = od; bj = oj; }
    }
    return bj;
}

// The nearest of all centroids for sixteen points a wave, lane (g, c) as in nearest_exact, which decides the near ties.  The same in
// a point's four lanes.
struct Decided {
    int id;
    float score, other;      // those of an AssignState
};
template <typename Points, typename IdOf>
__device__ __forceinline__ Decided nearest_of_all(const Points& X, int t, const unsigned char* rows_lds, uint32_t lds0, uint32_t ci0,
                                                  int k, float c2max, IdOf id_of)
{
    const int lane = lane_id(), c = lane & 15, g = lane >> 4;
    const int ntiles = (k + kRowTile - 1) / kRowTile;
    bf16x8_t x[4];
    float n2 = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const uint4 w = X.piece(t, 4 * ks + g);
        x[ks] = __builtin_bit_cast(bf16x8_t, w);
        n2 = dot2_bf16(w.x, w.x, n2);
        n2 = dot2_bf16(w.y, w.y, n2);
        n2 = dot2_bf16(w.z, w.z, n2);
        n2 = dot2_bf16(w.w, w.w, n2);
    }
    n2 += __shfl_xor(n2, 16, 64);
    n2 += __shfl_xor(n2, 32, 64);
    const uint32_t at = lds0 + (uint32_t)(c * 256 + ((g ^ c) & 3) * 16), turn = (uint32_t)((c >> 2) * 64);
    float best = -INFINITY, second = -INFINITY;
    int place = 0;
    for (int tile = 0; tile < ntiles; tile += 4) {
        f32x4_t s[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int tl = min(tile + r, ntiles - 1);
            s[r] = *reinterpret_cast<lds_four*>((uintptr_t)(ci0 + (uint32_t)((tl * kRowTile + 4 * g) * 4)));
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16x8_t f = *reinterpret_cast<lds_frag*>((uintptr_t)(at + (uint32_t)(tl * kRowTile * 256) + ((uint32_t)(64 * ks) ^ turn)));
                s[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, x[ks], s[r], 0, 0, 0);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (tile + r >= ntiles) continue;            // (uniform)
                second = fmaxf(second, fminf(best, s[r][i]));
                place = s[r][i] > best ? (tile + r) * kRowTile + 4 * g + i : place;
                best = fmaxf(best, s[r][i]);
            }
    }
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
        const float ob = __shfl_xor(best, off, 64), os = __shfl_xor(second, off, 64);
        const int op = __shfl_xor(place, off, 64);
        second = fmaxf(fmaxf(second, os), fminf(best, ob));
        place = ob > best ? op : place;                      // (equal ones are nearer than the margin)
        best = fmaxf(best, ob);
    }
    const float margin = near_margin(fmaxf(n2, c2max)) + fabsf(best) * (1.0f / 65536.0f);
    const bool near = !(best - second > margin);
    Decided d{id_of(min(place, k - 1)), kept_score(near, best, margin), near ? best : second};
    if (__any(near)) {
        const int id = nearest_exact(X, t, rows_lds, lds0, ci0, k, c2max, true, best, id_of);
        if (near) d.id = id;
    }
    return d;
}

// The chunk a wave takes next: the first that no wave has, `first` the one behind those the waves start with.  (In turn, the waves of a
// workgroup came to the barrier behind the chunks up to 40 us apart.)
__device__ __forceinline__ int next_chunk(int* ticket, int first)
{
    int t = 0;
    if (lane_id() == 0) t = atomicAdd(ticket, 1);
    return first + __builtin_amdgcn_readfirstlane(t);
}

template <int kW>
__global__ __launch_bounds__(64 * kW, 4) void assign_resident_kernel(const uint16_t* __restrict__ X, long long x_unit_rows,
                                                                    const int32_t* __restrict__ blocks,
                                                                    const uint16_t* __restrict__ C, long long c_unit_rows,
                                                                    int32_t* __restrict__ assign, long long assign_stride,
                                                                    int32_t* __restrict__ amb_list, long long list_stride,
                                                                    int32_t* __restrict__ cnt_next, int cnt_stride, int k_cap,
                                                                    const MoveMarks mv, const AssignState st)
{
    extern __shared__ __align__(256) unsigned char rows_lds[];    // [k_cap][256 bytes], then [k_cap] -|c|^2/2
    __shared__ float wave_c2max[kW];
    __shared__ int32_t near_list[kNearCap];                       // points for the exact pass, the first of them,
    __shared__ float near_best[kNearCap];                         // and their best scores
    __shared__ int near_n, ticket;
    const int u = blockIdx.z, b = blockIdx.y;
    // (this kernel leaves the counters of the other one alone; the next assignment step finds them zero all the same)
    if (b == 0 && blockIdx.x == 0)
        for (int i = threadIdx.x; i < cnt_stride; i += 64 * kW) cnt_next[u * cnt_stride + i] = 0;
    const int x0 = blocks[4 * b + 0], x1 = blocks[4 * b + 1], k0 = blocks[4 * b + 2];
    const int k1 = min(blocks[4 * b + 3], k0 + k_cap);            // (the launch guarantees the block has no more)
    const int all_chunks = (x1 - x0 + 63) / 64;
    const int per = (all_chunks + (int)gridDim.x - 1) / (int)gridDim.x;
    const int chunk0 = (int)blockIdx.x * per, chunk1 = min(chunk0 + per, all_chunks);
    if (chunk0 >= chunk1) return;
    if (mv.marks && blockIdx.x == 0 && threadIdx.x == 0) mv.moved_now[u * cnt_stride + b] = 0;
    if (unchanged(mv, u, b, cnt_stride)) {
        keep_chunks(mv, u, b, x0, x1, chunk0, chunk1, assign, assign_stride);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const PointsInMemory X_u{reinterpret_cast<const unsigned char*>(X + (long long)u * x_unit_rows * kHeadDim)};
    float* c_init = reinterpret_cast<float*>(rows_lds + k_cap * 256);

    // ---- the block's centroids: 16 lanes per row, rows past the last centroid are zeros that can never win ----
    const int ntiles = (k1 - k0 + kRowTile - 1) / kRowTile;
    float c2max = 0.f;
    {
        const uint16_t* Cu = C + (long long)u * c_unit_rows * kHeadDim;
        for (int e = tid; e < ntiles * kRowTile * 16; e += 64 * kW) {
            const int row = e >> 4, seg = e & 15;
            const bool exists = k0 + row < k1;
            uint4 w = make_uint4(0, 0, 0, 0);
            if (exists) w = reinterpret_cast<const uint4*>(Cu + (long long)(k0 + row) * kHeadDim)[seg];
            c2max = fmaxf(c2max, place_centroid(rows_lds, c_init, row, seg, w, exists));
        }
    }
    c2max = wave_max_f32(c2max);
    if (lane == 0) wave_c2max[wave] = c2max;
    if (tid == 0) near_n = ticket = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kW; ++w) c2max = fmaxf(c2max, wave_c2max[w]);

    int32_t* assign_u = assign + u * assign_stride;
    const int32_t* old_u = mv.old_ids + u * assign_stride;
    unsigned long long* marks = mv.marks + u * mv.stride + first_mark(x0, b);
    int32_t* more = amb_list + u * list_stride + x0 + chunk0 * 64;     // the others: as many entries as this workgroup has points
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)rows_lds;
#pragma unroll 1
    for (int chunk = chunk0 + wave; chunk < chunk1; chunk = next_chunk(&ticket, chunk0 + kW)) {
        const int t = x0 + chunk * 64 + lane;
        int old = 0;
        if (mv.marks) old = old_u[min(t, x1 - 1)];
        const Nearest r = nearest_of_chunk(X_u, x0 + chunk * 64, x1 - 1, lds0, lds0 + k_cap * 256, ntiles, c2max);
        if (mv.marks) {
            const unsigned long long marked = __ballot(t < x1 && (r.near || old != k0 + r.j));
            if (lane == 0) marks[chunk] = marked;
        }
        if (t < x1) {
            if (st.scores) st.scores[u * st.stride + t] = make_float2(kept_score(r.near, r.best, near_margin_of_best(r.m, r.best)), r.near ? r.best : r.second);
            if (r.near) {
                const int pos = atomicAdd(&near_n, 1);
                if (pos < kNearCap) {
                    near_list[pos] = t;
                    near_best[pos] = r.best;
                } else {
                    more[pos] = t;
                }
            } else {
                assign_u[t] = k0 + r.j;
            }
        }
    }
    __syncthreads();
    // ---- near ties: here, where the centroids are, instead of in a launch that fetches them for every point ----
    const int n = near_n;
    for (int e0 = wave * 16; e0 < n; e0 += kW * 16) {
        const int e = min(e0 + (lane_id() & 15), n - 1);
        const int t = e < kNearCap ? near_list[e] : more[e];
        const int j = nearest_exact(X_u, t, rows_lds, lds0, lds0 + k_cap * 256, k1 - k0, c2max, e0 < kNearCap, e < kNearCap ? near_best[e] : 0.f,
                                    [](int place) { return place; });
        if (lane_id() < 16) assign_u[t] = k0 + j;
    }
}

// The same step where the one before has left the scores it found (AssignState): a centroid that has not changed since scores
// what it did, so the points have to be compared with the changed ones only.  Of a point there is the score of its cluster's
// centroid, s, and a bound on the scores of all others, r >= what any of them scored (of a near tie, whose best score may be another's: s a margin below it, r that score).  With b the best and b2 the second best score
// among the changed centroids (its own among them if that changed):
//   - b is ahead of b2 and of r (and of s, if its own has not changed) by more than the margin: b's centroid is the one;
//   - its own has not changed and s is ahead of b by more than the margin: it keeps its cluster, which won the comparison with
//     the unchanged ones before, exactly where that was close;
//   - otherwise it goes onto a list and is compared with all centroids afterwards (nearest_of_all).
// The margins are those of two scores of one step (mp_margin.h): an older score that is compared as a centroid's own has the error of
// that centroid, which is still one of the block, and the largest |c|^2 is taken over all of them.
// 2048 blocks of 8192 keys, 256 centroids: 80 to 16 per cent of the centroids change in iterations 4 to 10, 3 to 0.5 per
// cent of the points go onto the list, and a launch takes 1.2 to 0.99 ms (compared with all: 1.13 to 1.29, by the clock it gets).  Bound by
// the keys it reads all the same: 0.81 ms without a single product, 0.93 with the points' ids and scores.  32 such blocks (of which 30 to 1 per cent
// of the centroids change): 34 to 18.5 us, all 33; there a launch without products takes 16, and what a workgroup adds is the chain
// of a point on its list, 10 us.
// The changed centroids stand in front; the others' -|c|^2/2 is one that never wins while the points are compared with the changed
// ones, tile by tile of sixteen.
template <int kW>
__global__ __launch_bounds__(64 * kW, 4) void assign_changed_kernel(const uint16_t* __restrict__ X, long long x_unit_rows,
                                                                   const int32_t* __restrict__ blocks,
                                                                   const uint16_t* __restrict__ C, long long c_unit_rows,
                                                                   int32_t* __restrict__ assign, long long assign_stride,
                                                                   int32_t* __restrict__ amb_list, long long list_stride,
                                                                   int32_t* __restrict__ cnt_next, int cnt_stride, int k_cap,
                                                                   const MoveMarks mv, const AssignState st)
{
    extern __shared__ __align__(256) unsigned char rows_lds[];    // [k_cap][256 bytes], [k_cap] -|c|^2/2, the same for changed ones only,
    float* c_init = reinterpret_cast<float*>(rows_lds + k_cap * 256);
    float* c_now = c_init + k_cap;
    uint16_t* ids = reinterpret_cast<uint16_t*>(c_now + k_cap);   // [k_cap] the centroid at a place,
    uint16_t* places = ids + k_cap;                               // [k_cap] the place of a centroid
    __shared__ float wave_c2max[kW];
    __shared__ int wave_changed[kW];
    __shared__ int32_t list[kNearCap];                            // points to be compared with all centroids, the first of them
    __shared__ int list_n, ticket;
    const int u = blockIdx.z, b = blockIdx.y;
    // (the counters of the other kernels, as in assign_resident_kernel)
    if (b == 0 && blockIdx.x == 0)
        for (int i = threadIdx.x; i < cnt_stride; i += 64 * kW) cnt_next[u * cnt_stride + i] = 0;
    const int x0 = blocks[4 * b + 0], x1 = blocks[4 * b + 1], k0 = blocks[4 * b + 2];
    const int k = min(blocks[4 * b + 3] - k0, k_cap);             // (the launch guarantees the block has no more)
    const int all_chunks = (x1 - x0 + 63) / 64;
    const int per = (all_chunks + (int)gridDim.x - 1) / (int)gridDim.x;
    const int chunk0 = (int)blockIdx.x * per, chunk1 = min(chunk0 + per, all_chunks);
    if (chunk0 >= chunk1) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) mv.moved_now[u * cnt_stride + b] = 0;
    if (unchanged(mv, u, b, cnt_stride)) {
        keep_chunks(mv, u, b, x0, x1, chunk0, chunk1, assign, assign_stride);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const PointsInMemory X_u{reinterpret_cast<const unsigned char*>(X + (long long)u * x_unit_rows * kHeadDim)};

    // ---- the block's centroids: asked for in the order of their ids, put in their places once it is known which have changed ----
    const int ntiles = (k + kRowTile - 1) / kRowTile;
    constexpr int kPieces = (kW == 8 ? kChangedTwiceK : kResidentMaxK) * 16 / (64 * kW);      // 16-byte pieces of a thread
    uint4 w[kPieces];
    const uint4* Cu = reinterpret_cast<const uint4*>(C + ((long long)u * c_unit_rows + k0) * kHeadDim);
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int e = tid + i * 64 * kW;
        if (i * 64 * kW < k * 16) w[i] = Cu[min(e, k * 16 - 1)];
    }
    const bool mine = tid < k && st.changed[u * st.changed_stride + k0 + tid] != 0;
    const unsigned long long which = __ballot(mine);
    if (lane == 0) wave_changed[wave] = __popcll(which);
    if (tid == 0) list_n = ticket = 0;
    __syncthreads();
    int n_changed = 0, before = 0;
#pragma unroll
    for (int i = 0; i < kW; ++i) {
        const int c = wave_changed[i];
        before += i < wave ? c : 0;
        n_changed += c;
    }
    if (tid < k) {
        const int rank = before + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(which >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)which, 0u));
        const int place = mine ? rank : n_changed + tid - rank;
        ids[place] = (uint16_t)tid;
        places[tid] = (uint16_t)place;
    }
    __syncthreads();
    float c2max = 0.f;
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int e = tid + i * 64 * kW, row = e >> 4, seg = e & 15;
        if (row < ntiles * kRowTile) {
            const bool exists = row < k;
            const int place = exists ? places[row] : row;
            const float s = place_centroid(rows_lds, c_init, place, seg, exists ? w[i] : make_uint4(0, 0, 0, 0), exists);
            if (seg == 0) c_now[place] = place < n_changed ? -0.5f * s : kNoCentroid;
            c2max = fmaxf(c2max, s);
        }
    }
    c2max = wave_max_f32(c2max);
    if (lane == 0) wave_c2max[wave] = c2max;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kW; ++i) c2max = fmaxf(c2max, wave_c2max[i]);

    int32_t* assign_u = assign + u * assign_stride;
    const int32_t* old_u = mv.old_ids + u * assign_stride;
    float2* scores_u = st.scores + u * st.stride;
    unsigned long long* marks = mv.marks + u * mv.stride + first_mark(x0, b);
    int32_t* more = amb_list + u * list_stride + x0 + chunk0 * 64;     // the others: as many entries as this workgroup has points
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)rows_lds;
    const uint32_t ci0 = lds0 + (uint32_t)(k_cap * 256);
    const int tiles_changed = (n_changed + kRowTile - 1) / kRowTile;
#pragma unroll 1
    for (int chunk = chunk0 + wave; chunk < chunk1; chunk = next_chunk(&ticket, chunk0 + kW)) {
        const int t = x0 + chunk * 64 + lane, tc = min(t, x1 - 1);
        const int old = old_u[tc];
        const float2 was = scores_u[tc];
        const Nearest r = nearest_of_chunk(X_u, x0 + chunk * 64, x1 - 1, lds0, ci0 + (uint32_t)(k_cap * 4), tiles_changed, c2max);
        const bool own_changed = (int)places[old - k0] < n_changed;
        const float others = fmaxf(own_changed ? was.y : fmaxf(was.x, was.y), r.second);
        const bool won = r.best - others > near_margin_of_best(r.m, r.best);
        const bool kept = !won && !own_changed && was.x - r.best > near_margin_of_best(r.m, was.x);
        const int id = won ? k0 + ids[r.j] : old;
        const unsigned long long marked = __ballot(t < x1 && (id != old || !(won || kept)));
        if (lane == 0) marks[chunk] = marked;
        if (t < x1) {
            if (won || kept) {
                assign_u[t] = id;
                if (won || r.best > was.y) scores_u[t] = won ? make_float2(r.best, others) : make_float2(was.x, r.best);
            } else {
                const int pos = atomicAdd(&list_n, 1);
                if (pos < kNearCap) list[pos] = t;
                else more[pos] = t;
            }
        }
    }
    __syncthreads();
    const int n = list_n;
    for (int e0 = wave * 16; e0 < n; e0 += kW * 16) {
        const int e = min(e0 + (lane_id() & 15), n - 1);
        const int t = e < kNearCap ? list[e] : more[e];
        const Decided d = nearest_of_all(X_u, t, rows_lds, lds0, ci0, k, c2max, [&](int place) { return (int)ids[place]; });
        if (lane_id() < 16) {
            assign_u[t] = k0 + d.id;
            scores_u[t] = make_float2(d.score, d.other);
        }
    }
}

template <typename Kernel>
hipError_t launch_resident(Kernel kernel, int waves, int bytes_per_row, bool& configured, const uint16_t* X, long long x_unit_rows,
                           const int32_t* blocks_dev, int nb, int max_pts, int max_k, int U, const uint16_t* C, long long c_unit_rows,
                           int32_t* assign, long long assign_stride, int32_t* amb_list, long long list_stride, int32_t* cnt_next,
                           int cnt_stride, const MoveMarks& mv, const AssignState& st, hipStream_t s)
{
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           kResidentMaxK * bytes_per_row);
        if (e != hipSuccess) return e;
        configured = true;
    }
    const int k_cap = (max_k + kRowTile - 1) / kRowTile * kRowTile;
    // workgroups per (block, unit): one round of resident workgroups where they fit it, else at least four rounds, so
    // that the last one weighs little.  With few pairs a workgroup may have a single chunk, for one of its waves: the
    // chip is idle otherwise, and its points' exact decisions are shared by all waves.  (A chunk a wave at least: 8192 points
    // x 512 centroids, 1 / 8 units, 338 / 456 us a build of five iterations against 264 / 397; the same with all keys
    // equal, every point decided exactly, 21.4 / 22.1 ms against 4.9 / 8.2.)
    const long long kSlots = 4096 / waves;                       // sixteen waves on each of 256 compute units
    const long long groups = (long long)nb * U;
    const int chunks = (max_pts + 63) / 64;
    const long long want = groups <= kSlots ? kSlots / groups : (4 * kSlots + groups - 1) / groups;
    const int gx = (int)std::max<long long>(1, std::min<long long>(chunks, want));
    hipLaunchKernelGGL(kernel, dim3(gx, nb, U), dim3(64 * waves), (size_t)k_cap * bytes_per_row, s, X, x_unit_rows,
                       blocks_dev, C, c_unit_rows, assign, assign_stride, amb_list, list_stride, cnt_next, cnt_stride, k_cap, mv, st);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// The coarse level of a range in one launch (Sec. 3.4): all Lloyd iterations over a block's fine centroids, the new
// order of the fine clusters, and the rows of the centroid tables that go with it.  One workgroup per (block, unit): a
// block has some hundred points and some tens of centroids, which fit one compute unit, and every step of an iteration is a
// few microseconds of latency when it is a launch of its own (assignment, exact pass, member lists, means: 30 us for 32
// (block, unit) pairs, times ten iterations).  Here an iteration is four barriers, and the
// first that moves no point ends them (the rest would repeat it); the decisions and sums are those of the
// separate kernels: near ties decided in fp64 as defined, members summed in ascending order in fp64, one rounding; only
// clusters of which a point has come or gone are summed again.
// Bound by the latency of one pair's chain.  So the points stand in LDS where they fit it beside the centroids (kInLds: rows for the products, the
// exact distances and the sums without a trip to memory), and a wave takes sixteen of them (a pair has some four chunks of 64 for
// its sixteen waves) and decides their near ties itself, with half the registers: 32 pairs of 256 points, 16 centroids and ten
// iterations 103 -> 81 us, 2048 pairs 810 -> 530; 64 pairs, three iterations 49 -> 37 us.  (Chunks of 64 points with a list of near
// ties behind a barrier, points in LDS: 85, 528 and 42 us.)
// ------------------------------------------------------------------------------------------------
template <int kW, bool kInLds>
__global__ __launch_bounds__(64 * kW, 4) void coarse_level_kernel(const CoarseLevel p)
{
    extern __shared__ __align__(256) unsigned char rows_lds[];   // [k_cap][256 bytes], kInLds: [n_cap][256 bytes] the points, [k_cap] -|c|^2/2, then:
    unsigned char* points_lds = rows_lds + p.k_cap * 256;
    float* c_init = reinterpret_cast<float*>(points_lds + (kInLds ? p.n_cap * 256 : 0));
    uint16_t* asg = reinterpret_cast<uint16_t*>(c_init + p.k_cap);    // [n_cap] cluster of each point
    uint16_t* order = asg + p.n_cap;                                  // [n_cap] points, cluster after cluster
    __shared__ int count[kLevelMaxK], moved;
    __shared__ bool touched[kLevelMaxK];                              // a point has come or gone
    __shared__ float wave_c2max[kW];
    const int b = blockIdx.x, u = blockIdx.y;
    const int x0 = p.blocks[4 * b + 0], n = p.blocks[4 * b + 1] - x0, k0 = p.blocks[4 * b + 2], k = p.blocks[4 * b + 3] - k0;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint4* Xb = reinterpret_cast<const uint4*>(p.X) + ((long long)u * p.x_unit_rows + x0) * 16;
    uint4* Ku = reinterpret_cast<uint4*>(p.Kc) + (long long)u * p.tab_rows * 16;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)rows_lds;
    const uint32_t ci0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)c_init;
    const int ntiles = (k + kRowTile - 1) / kRowTile;
    const int chunks = (n + 63) / 64;
    using Points = std::conditional_t<kInLds, PointsInLds, PointsInMemory>;
    const Points X{kInLds ? points_lds : reinterpret_cast<const unsigned char*>(Xb)};
    // one row by a wave, a dword a lane
    auto row_dword = [&](int t) {
        if constexpr (kInLds) return *reinterpret_cast<const uint32_t*>(points_lds + t * 256 + (((lane >> 2) ^ t) & 15) * 16 + (lane & 3) * 4);
        else return reinterpret_cast<const uint32_t*>(Xb)[(long long)t * 64 + lane];
    };

    // ---- first centroids: the stored ones of old clusters, seeds for the others; the points ----
    float c2max = 0.f;
    for (int e = tid; e < ntiles * kRowTile * 16; e += 64 * kW) {
        const int row = e >> 4, seg = e & 15, j = k0 + row;
        uint4 w = make_uint4(0, 0, 0, 0);
        if (row < k) {
            if (j < p.old_end) w = Ku[(long long)(p.fcap + j) * 16 + seg];
            else w = Xb[((long long)(p.seed_x0 < 0 ? 0 : p.seed_x0 - x0) + p.seeds[u * p.seed_stride + j]) * 16 + seg];
        }
        c2max = fmaxf(c2max, place_centroid(rows_lds, c_init, row, seg, w, row < k));
    }
    if constexpr (kInLds)
        for (int e = tid; e < n * 16; e += 64 * kW) {
            const int t = e >> 4, seg = e & 15;
            *reinterpret_cast<uint4*>(points_lds + t * 256 + ((seg ^ t) & 15) * 16) = Xb[e];
        }
    c2max = wave_max_f32(c2max);
    if (lane == 0) wave_c2max[wave] = c2max;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kW; ++w) c2max = fmaxf(c2max, wave_c2max[w]);

    for (int it = 0; it < p.iters; ++it) {
        if (tid == 0) moved = 0;
        for (int j = tid; j < k; j += 64 * kW) touched[j] = it == 0;
        __syncthreads();
        // ---- nearest centroid of every point, sixteen a wave: a pair has few chunks of 64, and the wave that finds a near tie decides it ----
        for (int t0 = wave * 16; t0 < n; t0 += kW * 16) {
            const int t = t0 + (lane & 15);
            const Decided d = nearest_of_all(X, min(t, n - 1), rows_lds, lds0, ci0, k, c2max, [](int place) { return place; });
            if (lane < 16 && t < n && (it == 0 || asg[t] != d.id)) {
                if (it > 0) touched[asg[t]] = touched[d.id] = true;
                asg[t] = (uint16_t)d.id;
                moved = 1;
            }
        }
        __syncthreads();
        if (moved == 0) break;        // the same assignment as before: the same centroids, and so in every iteration after it
        // ---- the clusters of which a point has come or gone: their members, one wave a cluster that finds them 64 at a time ----
        for (int j = wave; j < k; j += kW) {
            if (!touched[j]) continue;
            int m = 0;
            for (int ch = 0; ch < chunks; ++ch) {
                const int t = ch * 64 + lane;
                m += __popcll(__ballot(t < n && asg[t] == j));
            }
            if (lane == 0) count[j] = m;
        }
        __syncthreads();
        for (int j = wave; j < k; j += kW) {
            if (!touched[j]) continue;
            int pos = 0;                             // points of the clusters before this one
            for (int i = lane; i < j; i += 64) pos += count[i];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) pos += __shfl_xor(pos, off, 64);
            const int m = count[j];
            // this wave places the cluster's points, in ascending order, and sums their rows
            const int p0 = pos;
            for (int ch = 0; ch < chunks; ++ch) {
                const int t = ch * 64 + lane;
                const unsigned long long mine = __ballot(t < n && asg[t] == j);
                if ((mine >> lane) & 1ull) order[pos + __popcll(mine & ((1ull << lane) - 1ull))] = (uint16_t)t;
                pos += __popcll(mine);
            }
            wave_lds_sync();
            double a0 = 0.0, a1 = 0.0;
            for (int base = 0; base < m; base += 64) {
                const int nm = min(m - base, 64);
                const int member = lane < nm ? order[p0 + base + lane] : 0;
                constexpr int kBatch = 16;          // rows in flight (a cluster's time is its number of trips to memory)
                for (int q0 = 0; q0 < nm; q0 += kBatch) {
                    uint32_t w[kBatch];
#pragma unroll
                    for (int q = 0; q < kBatch; ++q) w[q] = row_dword(__builtin_amdgcn_readlane(member, min(q0 + q, nm - 1)));
#pragma unroll
                    for (int q = 0; q < kBatch; ++q) {
                        if (q0 + q < nm) {
                            a0 += (double)bf16lo_to_f32(w[q]);
                            a1 += (double)bf16hi_to_f32(w[q]);
                        }
                    }
                }
            }
            // new centroid (an empty cluster keeps its own), its place in LDS: dims 2 lane, 2 lane + 1
            if (m > 0) {
                const double den = (double)m;
                const uint32_t row = (uint32_t)f64_to_bf16_rne(a0 / den) | ((uint32_t)f64_to_bf16_rne(a1 / den) << 16);
                *(reinterpret_cast<uint32_t*>(rows_lds + j * 256 + (((lane >> 2) ^ j) & 15) * 16) + (lane & 3)) = row;
                float s = dot2_bf16(row, row, 0.f);
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
                if (lane == 0) c_init[j] = -0.5f * s;
            }
        }
        __syncthreads();
        c2max = 0.f;
        for (int j = lane; j < k; j += 64) c2max = fmaxf(c2max, -2.0f * c_init[j]);
        c2max = wave_max_f32(c2max);
    }
    // ---- the new order (that of the last iteration has holes where clusters kept their members) ----
    __syncthreads();
    for (int j = wave; j < k; j += kW) {
        int pos = 0;
        for (int i = lane; i < j; i += 64) pos += count[i];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) pos += __shfl_xor(pos, off, 64);
        for (int ch = 0; ch < chunks; ++ch) {
            const int t = ch * 64 + lane;
            const unsigned long long mine = __ballot(t < n && asg[t] == j);
            if ((mine >> lane) & 1ull) order[pos + __popcll(mine & ((1ull << lane) - 1ull))] = (uint16_t)t;
            pos += __popcll(mine);
        }
    }
    __syncthreads();
    // ---- list position -> old fine id, old -> new id, parents, and the rows of the tables ----
    const int at0 = x0 - p.f0;
    for (int i = tid; i < n; i += 64 * kW) {
        const int t = order[i];
        p.plist[u * p.list_stride + at0 + i] = x0 + t;
        p.newid[u * p.list_stride + x0 + t] = x0 + i;
        p.cof[u * p.list_stride + x0 + i] = k0 + asg[t];
    }
    for (int e = tid; e < n * 16; e += 64 * kW) {
        const int i = e >> 4, seg = e & 15;
        Ku[(long long)(x0 + i) * 16 + seg] = X.piece(order[i], seg);
    }
    for (int e = tid; e < k * 16; e += 64 * kW) {
        const int j = e >> 4, seg = e & 15;
        Ku[(long long)(p.fcap + k0 + j) * 16 + seg] = *reinterpret_cast<const uint4*>(rows_lds + j * 256 + ((seg ^ j) & 15) * 16);
    }
}

// Stage 2.  One wave per listed point, three passes over the block's centroids:
//   1. fp32 scores s_j = x.c_j - |c_j|^2/2 again (8 lanes per centroid, 16 dims each, sequential
//      fused multiply-adds: error far below the bound of stage 1), their maximum and max_j |c_j|^2;
//   2. every centroid whose score (kept in LDS, or computed once more for blocks with more than
//      kScoreCache centroids) is within the margin of the maximum is a candidate: the nearest
//      centroid in exact arithmetic, and everything tied with it, is among them;
//   3. the candidates' distances exactly as defined, one lane per candidate, fp64, no fused
//      multiply-adds, sum in index order; smallest distance wins, equal distances -> lowest index.
// More than kCandCap candidates (many coinciding centroids): every centroid is treated as one.
// grid = (nb, U, Z): the waves of a (block, unit) walk its list with stride 4 Z.  The list position
// is the slowest grid dimension, so that the few workgroups that have work are neighbours in
// dispatch order and spread over the whole chip.
constexpr int kCandCap = 64;
constexpr int kScoreCache = 2048;     // scores of pass 1 kept in LDS for pass 2 when the block has no more centroids

// |x - c|^2 in fp64, dims in index order, rounding after every operation
__device__ __forceinline__ double exact_distance(const uint16_t* xrow /*LDS*/, const uint16_t* crow /*global*/)
{
    double s = 0.0;
    const uint4* cp = reinterpret_cast<const uint4*>(crow);
    const uint4* xp = reinterpret_cast<const uint4*>(xrow);
#pragma unroll 2
    for (int i = 0; i < 16; ++i) {
        const uint4 cw = cp[i], xw = xp[i];
        const uint32_t c4[4] = {cw.x, cw.y, cw.z, cw.w}, x4[4] = {xw.x, xw.y, xw.z, xw.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double d0 = __dsub_rn((double)bf16lo_to_f32(x4[e]), (double)bf16lo_to_f32(c4[e]));
            const double d1 = __dsub_rn((double)bf16hi_to_f32(x4[e]), (double)bf16hi_to_f32(c4[e]));
            s = __dadd_rn(s, __dmul_rn(d0, d0));
            s = __dadd_rn(s, __dmul_rn(d1, d1));
        }
    }
    return s;
}

__global__ __launch_bounds__(256) void assign_recheck_kernel(const uint16_t* __restrict__ X, long long x_unit_rows,
                                                             const int32_t* __restrict__ blocks,
                                                             const uint16_t* __restrict__ C, long long c_unit_rows,
                                                             int32_t* __restrict__ assign, long long assign_stride,
                                                             const int32_t* __restrict__ amb_list, long long list_stride,
                                                             const int32_t* __restrict__ amb_cnt, int cnt_stride,
                                                             int32_t* __restrict__ cnt_next)
{
    __shared__ __align__(16) uint16_t xrow[4][kHeadDim];
    __shared__ int cand[4][kCandCap];
    __shared__ int ncand[4];
    __shared__ float sc_cache[4][kScoreCache];
    const int b = blockIdx.x, u = blockIdx.y;
    // the counters the next assignment step will count into (nobody reads them in this launch): all of the unit's
    if (b == 0 && blockIdx.z == 0)
        for (int i = threadIdx.x; i < cnt_stride; i += blockDim.x) cnt_next[u * cnt_stride + i] = 0;
    const int x0 = blocks[4 * b + 0], x1 = blocks[4 * b + 1], k0 = blocks[4 * b + 2], k1 = blocks[4 * b + 3];
    int n = amb_cnt[u * cnt_stride + b];
    if (n > x1 - x0) n = x1 - x0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = lane & 7, grp = lane >> 3;
    const uint16_t* Cu = C + (long long)u * c_unit_rows * kHeadDim;
    for (int e = (int)blockIdx.z * 4 + wave; e < n; e += (int)gridDim.z * 4) {
        const int t = amb_list[u * list_stride + x0 + e];
        const uint16_t* xg = X + ((long long)u * x_unit_rows + t) * kHeadDim;
        float xs[16];
        float x2 = 0.f;
        {
            const uint4 a = reinterpret_cast<const uint4*>(xg)[2 * sub], bq = reinterpret_cast<const uint4*>(xg)[2 * sub + 1];
            if (grp == 0) {
                reinterpret_cast<uint4*>(xrow[wave])[2 * sub] = a;
                reinterpret_cast<uint4*>(xrow[wave])[2 * sub + 1] = bq;
            }
            const uint32_t w[8] = {a.x, a.y, a.z, a.w, bq.x, bq.y, bq.z, bq.w};
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                xs[2 * q] = bf16lo_to_f32(w[q]);
                xs[2 * q + 1] = bf16hi_to_f32(w[q]);
                x2 = fmaf(xs[2 * q], xs[2 * q], x2);
                x2 = fmaf(xs[2 * q + 1], xs[2 * q + 1], x2);
            }
            x2 = sum8(x2);
        }
        // s_j and |c_j|^2 of four centroids j, j+8, j+16, j+24 by the 8 lanes of a group (every lane of
        // the group gets them); all eight row loads are issued before the first is used
        auto scores4 = [&](int j, float (&sc)[4], float (&cc)[4]) {
            uint4 a[4], bq[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int jr = (j + 8 * r < k1) ? j + 8 * r : k1 - 1;
                const uint4* cp = reinterpret_cast<const uint4*>(Cu + (long long)jr * kHeadDim);
                a[r] = cp[2 * sub];
                bq[r] = cp[2 * sub + 1];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t w[8] = {a[r].x, a[r].y, a[r].z, a[r].w, bq[r].x, bq[r].y, bq[r].z, bq[r].w};
                float dot = 0.f, c2 = 0.f;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const float lo = bf16lo_to_f32(w[q]), hi = bf16hi_to_f32(w[q]);
                    dot = fmaf(xs[2 * q], lo, dot);
                    dot = fmaf(xs[2 * q + 1], hi, dot);
                    c2 = fmaf(lo, lo, c2);
                    c2 = fmaf(hi, hi, c2);
                }
                dot = sum8(dot);
                c2 = sum8(c2);
                cc[r] = c2;
                sc[r] = (j + 8 * r < k1) ? fmaf(-0.5f, c2, dot) : -INFINITY;
            }
        };
        const bool cached = k1 - k0 <= kScoreCache;
        float best = -INFINITY, c2max = 0.f;
        for (int j = k0 + grp; j < k1; j += 32) {
            float sc[4], cc[4];
            scores4(j, sc, cc);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                best = fmaxf(best, sc[r]);
                c2max = fmaxf(c2max, cc[r]);        // (a clamped row repeats a real one)
                if (cached && sub == 0 && j + 8 * r < k1) sc_cache[wave][j + 8 * r - k0] = sc[r];
            }
        }
        best = wave_max_f32(best);
        c2max = wave_max_f32(c2max);
        const float thr = best - near_margin(fmaxf(x2, c2max));
        if (lane == 0) ncand[wave] = 0;
        wave_lds_sync();
        auto consider = [&](int j, float sc) {
            if (!(sc < thr)) {                       // also true for NaN
                const int pos = atomicAdd(&ncand[wave], 1);
                if (pos < kCandCap) cand[wave][pos] = j;
            }
        };
        if (cached) {
            for (int j = k0 + lane; j < k1; j += 64) consider(j, sc_cache[wave][j - k0]);
        } else {
            for (int j = k0 + grp; j < k1; j += 32) {
                float sc[4], cc[4];
                scores4(j, sc, cc);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (sub == 0 && j + 8 * r < k1) consider(j + 8 * r, sc[r]);
            }
        }
        wave_lds_sync();
        const int nc = ncand[wave];
        double bd = INFINITY;
        int bj = k0;
        if (nc <= kCandCap) {
            if (lane < nc) {
                const int j = cand[wave][lane];
                const double d = exact_distance(xrow[wave], Cu + (long long)j * kHeadDim);
                if (d < bd) { bd = d; bj = j; }
            }
        } else {
            for (int j = k0 + lane; j < k1; j += 64) {
                const double d = exact_distance(xrow[wave], Cu + (long long)j * kHeadDim);
                if (d < bd) { bd = d; bj = j; }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double od = __shfl_xor(bd, off, 64);
            const int oj = __shfl_xor(bj, off, 64);
            if (od < bd || (od == bd && oj < bj)) { bd = od; bj = oj; }
        }
        if (lane == 0) assign[u * assign_stride + t] = bj;
        wave_lds_sync();       // xrow / cand are reused by the next point
    }
}

}  // namespace

static size_t coarse_level_smem(int max_pts, int max_k, bool in_lds)
{
    const size_t k_cap = (size_t)(max_k + kRowTile - 1) / kRowTile * kRowTile, n_cap = (size_t)(max_pts + 3) / 4 * 4;
    return k_cap * 260 + n_cap * (in_lds ? 260 : 4);
}

template <int kW, bool kInLds>
static hipError_t launch_coarse_waves(const CoarseLevel& p, int nb, int U, size_t smem, hipStream_t s)
{
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&coarse_level_kernel<kW, kInLds>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           kInLds ? kCoarseLds : (int)coarse_level_smem(kLevelMaxPts, kLevelMaxK, false));
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL((coarse_level_kernel<kW, kInLds>), dim3(nb, U), dim3(64 * kW), smem, s, p);
    return hipGetLastError();
}

hipError_t launch_coarse_level(CoarseLevel p, int nb, int U, int max_pts, int max_k, hipStream_t s)
{
    if (nb <= 0 || U <= 0) return hipSuccess;
    if (max_pts < 1 || max_pts > kLevelMaxPts || max_k < 1 || max_k > kLevelMaxK || p.iters < 1) return hipErrorInvalidValue;
    p.k_cap = (max_k + kRowTile - 1) / kRowTile * kRowTile;
    p.n_cap = (max_pts + 3) / 4 * 4;
    // Sixteen waves where every pair has a compute unit of its own (a pair's time is what counts then: 104 against 132 us
    // for 32 pairs and ten iterations), else two workgroups of eight a compute unit (755 against 890 us for 2048 pairs), with the
    // points in LDS where two copies of them fit it.  (The four figures are from before the points stood there.)
    const size_t smem = coarse_level_smem(max_pts, max_k, false), with_points = coarse_level_smem(max_pts, max_k, true);
    static_assert((kLevelMaxPts + 64) * 260 <= kCoarseLds && (256 + 112) * 260 <= kCoarseLds, "whatever coarse_level_fits admits");
    if ((long long)nb * U <= 256) return with_points <= kCoarseLds ? launch_coarse_waves<16, true>(p, nb, U, with_points, s) : hipErrorInvalidValue;
    return with_points <= kCoarseLds / 2 ? launch_coarse_waves<8, true>(p, nb, U, with_points, s) : launch_coarse_waves<8, false>(p, nb, U, smem, s);
}

hipError_t launch_assign(const uint16_t* X, long long x_unit_rows, const int32_t* blocks_dev, int nb, int max_pts,
                         int max_k, int U, const uint16_t* C, long long c_unit_rows, int32_t* assign,
                         long long assign_stride, int32_t* amb_list, long long list_stride, int32_t* amb_cnt,
                         int32_t* amb_cnt_next, int cnt_stride, const MoveMarks& mv, const AssignState& st, hipStream_t s)
{
    if (nb <= 0 || max_pts <= 0 || U <= 0) return hipSuccess;
    if (nb > cnt_stride || U > 65535) return hipErrorInvalidValue;
    const int n_chunks = (max_pts + kPtsPerWg - 1) / kPtsPerWg;
    if (assign_is_resident(max_pts, max_k)) {
        // Two workgroups of eight waves a compute unit where two copies of the centroids fit its LDS, else one of sixteen.  Up to 256 blocks
        // of all units, sixteen take them in any case when all centroids are looked at (waves_for_blocks): a wave has a chunk or two there,
        // and half as many workgroups fetch the centroids -- but where that would leave a fifth of the waves out (129 to 170 blocks, 86 to
        // 102: one and two of the larger workgroups a block, three and five of the smaller), chunks and near ties wait for the waves there are:
        // 160 blocks of 8192 x 256 1759 / 1811, keys without clusters 2001 / 2047, few different keys 1868 / 2213; 96 1183 / 1189, 1408 / 1417, 1226 / 1314;
        // 129 of 1024 x 60, three iterations 194 / 198, 222 / 224, 238 / 257.
        // Elsewhere, builds of ten iterations (three of these steps), us, eight / sixteen waves, two runs each that differ by up to 0.5 %
        // (128 blocks: 1.3): 8 blocks of 8192 x 256 336 / 331, keys without clusters 601 / 593; 32 617 / 611 and 899 / 873; 64 885 / 872 and
        // 1095 / 1081; 72 1003 / 989 and 1222 / 1206; 104 1273 / 1263 and 1502 / 1492; 192 2119 / 2096 and 2300 / 2268; level at 256: 2499 /
        // 2502 and 2663 / 2682; 2048 19853 / 19933.  (Settled iterations keep eight: 32 blocks 644 / 651, 2048 19842 / 20140, keys without clusters 924 / 925; 64, the one gain, 1133 / 1111.)
        static bool configured[4] = {};
        auto go = [&](auto kernel, int waves, int bytes_per_row, bool& set) {
            return launch_resident(kernel, waves, bytes_per_row, set, X, x_unit_rows, blocks_dev, nb, max_pts, max_k, U, C, c_unit_rows,
                                   assign, assign_stride, amb_list, list_stride, amb_cnt_next, cnt_stride, mv, st, s);
        };
        if (st.changed)
            return max_k <= kChangedTwiceK ? go(assign_changed_kernel<8>, 8, 268, configured[0]) : go(assign_changed_kernel<16>, 16, 268, configured[1]);
        return max_k <= kResidentTwiceK && waves_for_blocks((long long)nb * U) == 8 ? go(assign_resident_kernel<8>, 8, 260, configured[2]) : go(assign_resident_kernel<16>, 16, 260, configured[3]);
    }
    hipLaunchKernelGGL(assign_mfma_kernel, dim3(n_chunks, nb, U), dim3(256), 0, s, X, x_unit_rows, blocks_dev, C,
                       c_unit_rows, assign, assign_stride, amb_list, list_stride, amb_cnt, cnt_stride, mv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int z = std::min(32, (max_pts + 3) / 4);      // (deeper grids only add workgroups that find nothing to do)
    hipLaunchKernelGGL(assign_recheck_kernel, dim3(nb, U, z), dim3(256), 0, s, X, x_unit_rows,
                       blocks_dev, C, c_unit_rows, assign, assign_stride, amb_list, list_stride, amb_cnt, cnt_stride,
                       amb_cnt_next);
    return hipGetLastError();
}

}  // namespace mp
