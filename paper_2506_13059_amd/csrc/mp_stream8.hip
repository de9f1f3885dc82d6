// Value pass over 8-bit rows on the matrix cores, for gfx950 (the layout of the rows: RowSource; mp_stream.hip has the scheme
// and the kernel for bf16 rows).
//
// A wave streams tiles of 32 rows: 128-byte code rows of keys and values go straight to LDS, sixteen bytes a lane and eight
// rows an instruction, and with them the rows' scales and their logit shares (q . centroid, from L2), in a ring of two tiles.
//   S = K Q^T      the codes of an A operand's lane are eight bytes; they become bf16 in registers (exact: four significant
//                  bits), two 16-row products of four steps; logit = S * key scale + the row's share
//   O += P V       P times the value scale, split into three bf16 parts as in mp_stream.hip; the codes of 32 rows of one dim
//                  come to a lane by the transposing 8-bit read (rows 4g .. 4g+3 and 16+4g .. 16+4g+3, as the scores lie)
//                  and become bf16 there: one product of 32 rows each of the eight groups of dims
// Bound by the memory system and its latency: two vector instructions a code pair are all that 8 bits cost, about 200 for 32
// rows; the vector-ALU kernel needs 420 for 16.
// Whole step, vector-ALU kernel -> here: 64 units, 3125 of 100003 keys and a tail of 139, 4 heads 54.7 -> 42.7 us; 64 x 4096, 8
// heads 67.3 -> 42.3 and 128 x 4096, 4 heads 64.3 -> 52.0 when they were measured (one and two heads: bytes_on_vector_alu in mp_plan.h).
#include "mp_stream_tiles.h"

namespace mp {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr int kTile8 = 32;                       // rows per tile
constexpr int kCodes = kTile8 * 128;             // bytes of a tile's keys (or values)
constexpr int kShares = kTile8 * 32;             // ... logit shares: columns 0 .. 3 of every row, then columns 4 .. 7
constexpr int kScales = kTile8 * 8;              // ... {key scale, value scale}
constexpr int kSlot8 = 2 * kCodes + kShares + kScales;
constexpr int kRing8 = 2 * kSlot8;               // per wave
constexpr int kStrips8 = 20 * kStrip;            // two strips of row numbers, two of cluster slots, the guest source's first
static_assert(kRing8 >= kRing && kStrips8 >= kStripBytes, "the other sources of a launch use the same space");
static_assert(4 * (kRing8 + kStrips8) <= 80 * 1024, "two workgroups a compute unit");

__device__ __forceinline__ bf16x8 widen_codes(u32x2 w)
{
    const bf16x2 v[4] = {__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w.x, 1.0f, false), __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w.x, 1.0f, true),
                         __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w.y, 1.0f, false), __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w.y, 1.0f, true)};
    return bf16x8{v[0].x, v[0].y, v[1].x, v[1].y, v[2].x, v[2].y, v[3].x, v[3].y};
}

// The weights of the rows' codes are probabilities times value scales, of any magnitude, and the lowest bit of a bf16 part is
// 2^-133 at best.  So from a scale below kSmallScale on a wave takes its weights, and the sums it has, kRaise times up, which
// leaves every part its bits down to the smallest values; a scale from kLargeScale on ends that (below it a sum of 2^24 rows
// taken up stays finite) and may be infinite.  A wave looks for such scales only where the index has had one (`unusual`, which the
// quantiser notes): a comparison a tile alone made launches over a tile or two 0.2 us longer.
constexpr float kRaise = 0x1p64f;
enum class Weights { ordinary, raised, large };
template <int G>
__device__ __forceinline__ void scale_sums(StreamState<G>& st, float by)
{
#pragma unroll
    for (int d = 0; d < 8; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            st.o[d][i] *= by;
            if constexpr (StreamState<G>::kThird) st.o3[d][i] *= by;
        }
}

// The same part of eight weights as tile_values takes of four probabilities, and their product with the rows.  Codes are finite, so
// a part of zero needs no floor; an infinite weight (`large`: there may be one) is its own part, every time.
template <int G>
__device__ __forceinline__ void tile_values8(StreamState<G>& st, const float (&p)[8], bool large, uint32_t v_addr, uint32_t mask1, uint32_t mask2)
{
    float x[2][4], y[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = p[4 * h + i];
            x[h][i] = v - __uint_as_float(__float_as_uint(v) & mask1);
            if constexpr (StreamState<G>::kThird) {
                const float r = v - __uint_as_float(__float_as_uint(v) & 0xffff0000u);
                y[h][i] = r - __uint_as_float(__float_as_uint(r) & 0xffff0000u);
            } else {
                x[h][i] = x[h][i] - __uint_as_float(__float_as_uint(x[h][i]) & mask2);
            }
        }
    }
    if (__builtin_expect(large, 0)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (p[i] != INFINITY) continue;
            x[i >> 2][i & 3] = INFINITY;
            if constexpr (StreamState<G>::kThird) y[i >> 2][i & 3] = INFINITY;
        }
    }
    auto operand = [&](const float (&z)[2][4]) {
        const u32x2 lo = __builtin_bit_cast(u32x2, upper_halves(z[0])), hi = __builtin_bit_cast(u32x2, upper_halves(z[1]));
        return __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
    };
    const bf16x8 a = operand(x);
    u32x2 v[8];
    const uint32_t a1 = v_addr ^ 16u, a2 = v_addr ^ 32u, a3 = v_addr ^ 48u, a4 = v_addr ^ 64u, a5 = v_addr ^ 80u, a6 = v_addr ^ 96u, a7 = v_addr ^ 112u;
    asm volatile("ds_read_b64_tr_b8 %0, %8\n\tds_read_b64_tr_b8 %1, %9\n\tds_read_b64_tr_b8 %2, %10\n\t"
                 "ds_read_b64_tr_b8 %3, %11\n\tds_read_b64_tr_b8 %4, %12\n\tds_read_b64_tr_b8 %5, %13\n\t"
                 "ds_read_b64_tr_b8 %6, %14\n\tds_read_b64_tr_b8 %7, %15\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                 : "v"(v_addr), "v"(a1), "v"(a2), "v"(a3), "v"(a4), "v"(a5), "v"(a6), "v"(a7)
                 : "memory");
    bf16x8 w[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) w[d] = widen_codes(v[d]);
#pragma unroll
    for (int d = 0; d < 8; ++d) st.o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w[d], st.o[d], 0, 0, 0);
    if constexpr (StreamState<G>::kThird) {
        const bf16x8 b = operand(y);
#pragma unroll
        for (int d = 0; d < 8; ++d) st.o3[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, w[d], st.o3[d], 0, 0, 0);
    }
}

// Listed 8-bit rows [w0, w1) through one wave (the counterpart of stream_tiles, whose comments on the pipeline hold here).
// The wave's sums are still zero.  unusual: whether a value scale may lie outside [kSmallScale, kLargeScale).
template <int G, typename Started>
__device__ __forceinline__ void stream_tiles8(StreamState<G>& st, const RowSource& S, const ValuePassParams& p, int u, bool unusual, int w0, int w1,
                                              uint32_t ring, uint32_t strips, Started started)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int head = c % G, part = c / G;                         // (columns beyond the last part repeat a head)
    const uint32_t mask1 = part >= 1 ? 0xffff0000u : 0u, mask2 = part >= 2 ? 0xffff0000u : 0u;
    const unsigned char* Kb = reinterpret_cast<const unsigned char*>(S.K) + (long long)u * S.unit_rows * 128;
    const unsigned char* Vb = reinterpret_cast<const unsigned char*>(S.V) + (long long)u * S.unit_rows * 128;
    const float* scales = S.row_scale + ((long long)u * S.unit_rows) * 2 + (lane & 1);
    const float* shares = S.slot_base + (long long)u * S.base_stride * 8 + 4 * (lane >> 5);
    const int32_t* rows = S.rows + (long long)u * S.rows_stride;
    const int32_t* slots = S.row_slot + (long long)u * S.rows_stride;
    bf16x8 q[4];
    {
        const uint4* qp = reinterpret_cast<const uint4*>(p.q + ((long long)u * G + head) * kHeadDim);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) q[ks] = __builtin_bit_cast(bf16x8, qp[4 * ks + g]);
    }
    // LDS layout of codes: row r at 128 r, its 16-byte chunk j at position j ^ (r / 2 mod 8) (conflict-free reads).
    // loads: instruction i covers rows 8i .. 8i+7, lane = 8 (row - 8i) + position
    const int lr = lane >> 3;
    const uint32_t k_addr = ring + (uint32_t)(c * 128 + (((g >> 1) ^ (c >> 1)) & 7) * 16 + (g & 1) * 8);           // ^ 32 ks, + 2048: rows 16 and up
    const int e = c >> 1, vr = e < 4 ? 4 * g + e : 12 + 4 * g + e;                                                 // (16 + 4 g + e - 4)
    const uint32_t v_addr = ring + kCodes + (uint32_t)(vr * 128 + ((vr >> 1) & 7) * 16 + (c & 1) * 8);            // ^ 16 d
    constexpr int kHalf = G > 5 ? (G + 1) / 2 : 8;                // (the scoring launch's columns: see fast_epilogue)
    const int col = head < kHalf ? head : 4 + head - kHalf;
    const uint32_t share_addr = ring + 2 * kCodes + (uint32_t)((col >> 2) * (kShares / 2) + (col & 3) * 4 + 4 * g * 16);
    const uint32_t scale_addr = ring + 2 * kCodes + kShares + (uint32_t)(4 * g * 8);
    const int n_tiles = (w1 - w0 + kTile8 - 1) / kTile8;

    auto load_strip = [&](int s) {           // row numbers and slots [w0 + 64 s, +64), clamped to the last row
        const int j = min(w0 + s * kStrip + lane, w1 - 1);
        load_to_lds<4, false>(rows + j, strips + (uint32_t)((s & 1) * 4 * kStrip));
        load_to_lds<4, false>(slots + j, strips + (uint32_t)((2 + (s & 1)) * 4 * kStrip));
    };
    long long off[4];                        // byte offsets of the code rows this lane loads for a tile
    int scale_row, slot;
    auto tile_rows = [&](int t) {
        const uint32_t at = strips + (uint32_t)((((t >> 1) & 1) * kStrip + (t & 1) * kTile8) * 4);
        const uint32_t a0 = at + 4u * lr, a1 = at + 4u * (lane >> 1), a2 = at + 4u * (2 * kStrip + (lane & 31));
        int r[4];
        asm volatile("ds_read_b32 %0, %6\n\tds_read_b32 %1, %6 offset:32\n\tds_read_b32 %2, %6 offset:64\n\tds_read_b32 %3, %6 offset:96\n\t"
                     "ds_read_b32 %4, %7\n\tds_read_b32 %5, %8\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(scale_row), "=&v"(slot)
                     : "v"(a0), "v"(a1), "v"(a2)
                     : "memory");
        if (t == n_tiles - 1) {              // (past the share's end a strip holds anything: the tile's first row instead)
            const int row0 = __builtin_amdgcn_readfirstlane(r[0]), slot0 = __builtin_amdgcn_readfirstlane(slot), left = w1 - w0 - t * kTile8;
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = 8 * i + lr < left ? r[i] : row0;
            scale_row = (lane >> 1) < left ? scale_row : row0;
            slot = (lane & 31) < left ? slot : slot0;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) off[i] = (long long)r[i] * 128 + (((lane & 7) ^ ((8 * i + lr) >> 1)) & 7) * 16;
    };
    auto slot_at = [&](int t) { return ring + (uint32_t)((t & 1) * kSlot8); };
    constexpr int kKeyLoads = 6;
    auto load_keys = [&](int t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) load_to_lds<16, true>(Kb + off[i], slot_at(t) + (uint32_t)(i * 1024));
        load_to_lds<16, false>(shares + (long long)slot * 8, slot_at(t) + 2 * kCodes);
        load_to_lds<4, false>(scales + (long long)scale_row * 2, slot_at(t) + 2 * kCodes + kShares);
    };
    auto load_values = [&](int t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) load_to_lds<16, true>(Vb + off[i], slot_at(t) + (uint32_t)(kCodes + i * 1024));
    };

    // K0 V0 K1 V1 K2 V2 ..., six instructions (codes, shares, scales) and four, two for a strip now and then.
    const bool single = n_tiles == 1;
    wait_vm<0>();
    tile_rows(0);
    if (n_tiles > kStrip / kTile8) load_strip(1);
    load_keys(0);
    load_values(0);
    started();
    if (!single) {
        tile_rows(1);
        load_keys(1);
        load_values(1);
        if (n_tiles > 2 * (kStrip / kTile8)) load_strip(2);      // (the first strip's numbers have all been read)
    }
    Weights weights = Weights::ordinary;     // (the same in all lanes)
    auto tile = [&](int t, auto ahead) {
        constexpr int kAhead = decltype(ahead)::value;            // how many tiles follow (two: two or more)
        const uint32_t half = (uint32_t)((t & 1) * kSlot8);
        wait_vm<kAhead == 0 ? 4 : 8 + kKeyLoads>();
        u32x2 k[2][4];
        u32x4 sc[4];
        float share[8];
        {
            const uint32_t a0 = k_addr + half, a1 = (k_addr ^ 32u) + half, a2 = (k_addr ^ 64u) + half, a3 = (k_addr ^ 96u) + half;
            asm volatile("ds_read_b64 %0, %20\n\tds_read_b64 %1, %21\n\tds_read_b64 %2, %22\n\tds_read_b64 %3, %23\n\t"
                         "ds_read_b64 %4, %20 offset:2048\n\tds_read_b64 %5, %21 offset:2048\n\tds_read_b64 %6, %22 offset:2048\n\t"
                         "ds_read_b64 %7, %23 offset:2048\n\t"
                         "ds_read_b128 %8, %24\n\tds_read_b128 %9, %24 offset:16\n\tds_read_b128 %10, %24 offset:128\n\t"
                         "ds_read_b128 %11, %24 offset:144\n\t"
                         "ds_read_b32 %12, %25\n\tds_read_b32 %13, %25 offset:16\n\tds_read_b32 %14, %25 offset:32\n\t"
                         "ds_read_b32 %15, %25 offset:48\n\tds_read_b32 %16, %25 offset:256\n\tds_read_b32 %17, %25 offset:272\n\t"
                         "ds_read_b32 %18, %25 offset:288\n\tds_read_b32 %19, %25 offset:304\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(k[0][0]), "=&v"(k[0][1]), "=&v"(k[0][2]), "=&v"(k[0][3]), "=&v"(k[1][0]), "=&v"(k[1][1]), "=&v"(k[1][2]),
                           "=&v"(k[1][3]), "=&v"(sc[0]), "=&v"(sc[1]), "=&v"(sc[2]), "=&v"(sc[3]), "=&v"(share[0]), "=&v"(share[1]),
                           "=&v"(share[2]), "=&v"(share[3]), "=&v"(share[4]), "=&v"(share[5]), "=&v"(share[6]), "=&v"(share[7])
                         : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(scale_addr + half), "v"(share_addr + half)
                         : "memory");
        }
        if constexpr (kAhead == 2) {
            tile_rows(t + 2);
            load_keys(t + 2);
        }
        float s[8], vs[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(widen_codes(k[h][ks]), q[ks], acc, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32x4 w = sc[2 * h + (i >> 1)];
                s[4 * h + i] = fmaf(acc[i], p.scale_log2e * __uint_as_float(i & 1 ? w.z : w.x), share[4 * h + i]);
                vs[4 * h + i] = __uint_as_float(i & 1 ? w.w : w.y);
            }
        }
        if constexpr (kAhead == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) s[i] = w0 + t * kTile8 + 16 * (i >> 2) + 4 * g + (i & 3) < w1 ? s[i] : -INFINITY;
        }
        float pr[8];
        tile_softmax<G>(st, s, pr);
        if (__builtin_expect(unusual, 0)) {
            float least = vs[0], most = vs[0];
#pragma unroll
            for (int i = 1; i < 8; ++i) {
                least = fminf(least, vs[i]);
                most = fmaxf(most, vs[i]);
            }
            const bool large = __any(most >= kLargeScale), small = __any(least < kSmallScale);
            const Weights now = large || weights == Weights::large ? Weights::large : small ? Weights::raised : weights;
            if (now != weights) scale_sums(st, now == Weights::raised ? kRaise : weights == Weights::raised ? 1.f / kRaise : 1.f);
            weights = now;
            if (weights == Weights::raised) {
#pragma unroll
                for (int i = 0; i < 8; ++i) vs[i] *= kRaise;
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) pr[i] *= vs[i];
        if constexpr (kAhead == 0) {         // (the rows past the end repeat the last one: nothing of them, whatever their scale)
#pragma unroll
            for (int i = 0; i < 8; ++i) pr[i] = w0 + t * kTile8 + 16 * (i >> 2) + 4 * g + (i & 3) < w1 ? pr[i] : 0.f;
        }
        wait_vm<kAhead == 2 ? 4 + 2 * kKeyLoads : kAhead * (4 + kKeyLoads)>();
        tile_values8<G>(st, pr, weights == Weights::large, v_addr + half, mask1, mask2);
        if constexpr (kAhead == 2) {
            load_values(t + 2);
            // the row numbers of tile t + 2, the last of its strip, have just been read: its slot takes the strip after next
            if ((t & 1) == 1 && ((t >> 1) + 3) * (kStrip / kTile8) < n_tiles) load_strip((t >> 1) + 3);
        }
    };
    int t = 0;
    for (; t + 2 < n_tiles; ++t) tile(t, std::integral_constant<int, 2>{});
    if (!single) tile(t++, std::integral_constant<int, 1>{});
    tile(t, std::integral_constant<int, 0>{});
    if (weights == Weights::raised) scale_sums(st, 1.f / kRaise);
}

// As value_stream_kernel; the selected keys, the launch's last source, are 8-bit rows, the centroid terms (src[0], which rides along) and the
// tail bf16 rows.  rows, slots, counts, rows_stride, chunk0, chunk_rows: the keys' source, n_terms: the number of the terms (null: none), as scalars
// of the launch, so that the first row numbers and the counts do not wait for the other arguments (whole
// step: 64 units, 3125 of 100003 keys and a tail 43.6 -> 42.7 us; 8 units x 4096 keys 24.1 -> 23.5; 32 units of 8 heads and a tail 36.7 -> 35.7).
template <int G>
__global__ __launch_bounds__(256, 2) void value_stream8_kernel(const int32_t* rows, const int32_t* slots, const int32_t* counts, const int32_t* n_terms,
                                                               int rows_stride, int n_units, int chunk0, int chunk_rows, const ValuePassParams p)
{
    constexpr int kWaves = 4;
    extern __shared__ __align__(256) unsigned char ring_lds[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)ring_lds;
    const uint32_t ring = lds0 + (uint32_t)(wave * kRing8), strips = lds0 + (uint32_t)(kWaves * kRing8 + wave * kStrips8);
    const uint32_t guest_strip = strips + 16 * kStrip;
    StreamShare w;
    w.chunk = blockIdx.x / n_units;
    const int u = w.u = blockIdx.x - w.chunk * n_units;
    const bool keys = w.chunk >= chunk0;     // (the others have rows of the tail)
    typedef const __attribute__((address_space(4))) int32_t constant_int;
    int counted = 0, unusual = 0, terms = 0;
    if (keys) {
        counted = ((constant_int*)counts)[u];
        unusual = ((constant_int*)counts)[n_units];
        if (n_terms) terms = ((constant_int*)n_terms)[u];
        const int first = (w.chunk - chunk0) * chunk_rows + wave * ((chunk_rows / kWaves + kTile - 1) / kTile * kTile);
        const long long at = (long long)u * rows_stride + min(first + (tid & 63), rows_stride - 1);
        load_to_lds<4, false>(rows + at, strips);
        load_to_lds<4, false>(slots + at, strips + 8 * kStrip);
    }
    touch_arguments(p);
    asm volatile("" ::"s"(counted), "s"(unusual), "s"(terms));
    const RowSource& S = p.src[keys ? p.n_sources - 1 : p.n_sources - 2];
    w.begin = (w.chunk - S.chunk0) * S.chunk_rows;
    w.end = min(w.begin + S.chunk_rows, keys ? min(counted, S.count_max) : S.count_max);
    const int wave_rows = (S.chunk_rows / kWaves + kTile - 1) / kTile * kTile;
    w.w0 = w.begin + wave * wave_rows;
    w.w1 = min(w.w0 + wave_rows, w.end);
    w.g0 = w.g1 = 0;
    if (n_terms && keys) {
        const long long n = min(terms, p.src[0].count_max), k = w.chunk - S.chunk0;
        w.g0 = (int)(n * k / S.n_chunks);
        w.g1 = (int)(n * (k + 1) / S.n_chunks);
    }
    const int per = ((w.g1 - w.g0 + kWaves - 1) / kWaves + 15) & ~15;
    w.a = w.g0 + wave * per;
    w.b = min(w.a + per, w.g1);
    float* part = p.partials + ((long long)u * p.chunks_per_unit + w.chunk) * G * kPartStride;
    if (w.w0 >= w.w1) nothing_on_its_way();  // (what was asked for early is in place before its space is used or given back)
    if (w.begin >= w.end && w.g0 >= w.g1) {
        if (tid < G) {
            part[tid * kPartStride + 0] = -INFINITY;
            part[tid * kPartStride + 1] = 0.f;
        }
        return;
    }
    StreamState<G> st;
    clear_state(st);
    auto guest = [&] { if (w.a < w.b) fetch_strip(p.src[0].rows, p.src[0], u, w.a, guest_strip); };
    if (w.w0 < w.w1) {
        if (keys) stream_tiles8<G>(st, S, p, u, unusual != 0, w.w0, w.w1, ring, strips, guest);
        else stream_tiles<G, false, false>(st, S, p, u, w.w0, w.w1, ring, strips, guest);
    } else {
        guest();
    }
    if (w.a < w.b) {
        take_guest_strip(guest_strip, strips);
        stream_tiles<G, true, true>(st, p.src[0], p, u, w.a, w.b, ring, strips, [] {});
    }
    combine_waves<G, kWaves>(st, reinterpret_cast<float*>(ring_lds), part);
}

template <int G>
hipError_t launch_stream8_g(const ValuePassParams& p, hipStream_t s)
{
    const long long blocks = (long long)p.n_units * p.chunks_per_unit;
    if (blocks <= 0) return hipSuccess;
    static bool configured = false;
    constexpr size_t smem = 4 * (kRing8 + kStrips8);
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&value_stream8_kernel<G>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    const RowSource& S = p.src[p.n_sources - 1];
    hipLaunchKernelGGL((value_stream8_kernel<G>), dim3((unsigned)blocks), dim3(256), smem, s, S.rows, S.row_slot, S.count_dev,
                       S.guest ? p.src[0].count_dev : nullptr, (int)S.rows_stride, p.n_units, S.chunk0, S.chunk_rows, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_value_stream8(const ValuePassParams& p, int G, hipStream_t s)
{
    // the terms, if they ride along, perhaps a tail, the selected keys
    if (p.n_sources < 1 || p.n_sources > 3) return hipErrorInvalidValue;
    const RowSource& S = p.src[p.n_sources - 1];
    const int tails = p.n_sources - 1 - (S.guest ? 1 : 0);
    if (!S.rows || !S.row_slot || !S.row_scale || !S.count_dev || S.row0 != 0 || S.rows_stride > 0x7fffffff || tails < 0 || tails > 1 ||
        (S.guest && (!p.src[0].scores || !p.src[0].count_dev || p.src[0].n_chunks != 0)) ||
        (tails == 1 && (p.src[p.n_sources - 2].rows || p.src[p.n_sources - 2].count_dev || p.src[p.n_sources - 2].row0 != 0)) || (tails == 0 && S.chunk0 != 0))
        return hipErrorInvalidValue;
    switch (G) {
        case 2: return launch_stream8_g<2>(p, s);
        case 3: return launch_stream8_g<3>(p, s);
        case 4: return launch_stream8_g<4>(p, s);
        case 5: return launch_stream8_g<5>(p, s);
        case 6: return launch_stream8_g<6>(p, s);
        case 7: return launch_stream8_g<7>(p, s);
        case 8: return launch_stream8_g<8>(p, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mp
