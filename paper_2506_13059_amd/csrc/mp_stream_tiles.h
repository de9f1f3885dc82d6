// Device code of the matrix-core value passes (mp_stream.hip: bf16 rows; mp_stream8.hip: 8-bit rows): one wave streaming a
// source of bf16 rows, the online softmax, the exact split of the probabilities, and the end of a workgroup.
#pragma once
#include <type_traits>

#include "mp_device.h"
#include "mp_internal.h"

namespace mp {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kTile = 16;                        // rows per tile
constexpr int kPiece = kTile * 256;              // bytes of a tile's keys (or values)
constexpr int kRing = 4 * kPiece;                // per wave: keys and values of two tiles
constexpr int kScores = 1024;                    // in the place of a tile's keys: ready-made logits (512 bytes of eight heads)
constexpr int kScoredRing = 2 * (kScores + kPiece);
constexpr int kStrip = 64;                       // row numbers fetched at a time
constexpr int kStripBytes = 12 * kStrip;         // per wave: two strips, and the first one of the launch's guest source

typedef __attribute__((address_space(3))) unsigned char lds_byte;

template <int kBytes, bool kOnce>
__device__ __forceinline__ void load_to_lds(const void* src, uint32_t lds_off)
{
    // (the LDS address is the same in all lanes; lane i's bytes go to it + kBytes * i)
    auto* dst = reinterpret_cast<__attribute__((address_space(3))) uint32_t*>((uintptr_t)lds_off);
    auto* from = (const __attribute__((address_space(1))) uint32_t*)src;
    if constexpr (kBytes == 16 && kOnce) __builtin_amdgcn_global_load_lds(from, dst, 16, 0, 2);     // (2: non-temporal)
    else if constexpr (kBytes == 16) __builtin_amdgcn_global_load_lds(from, dst, 16, 0, 0);
    else __builtin_amdgcn_global_load_lds(from, dst, 4, 0, 0);
}
template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// A wave without rows waits for its early loads.
__device__ __forceinline__ void nothing_on_its_way()
{
    __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0)
}
// Four row numbers, 16 bytes apart.
__device__ __forceinline__ void lds_read_rows(uint32_t a, int (&r)[4])
{
    asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:16\n\tds_read_b32 %2, %4 offset:32\n\t"
                 "ds_read_b32 %3, %4 offset:48\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
                 : "v"(a)
                 : "memory");
}

template <int G>
struct StreamState {
    static constexpr bool kThird = 3 * G > 16;          // third parts in products of their own
    f32x4 o[8];                                         // rows 4g+i = columns part * G + h, lane & 15 = dim of the 16
    f32x4 o3[kThird ? 8 : 1];
    float m, l;                                         // of this lane's column
};

// Online softmax of one tile's scores (rows 4g+i of this lane's column; eight scores: rows 16+4g+i, too) and the product
// with its value rows.
template <int G, int N>
__device__ __forceinline__ void tile_softmax(StreamState<G>& st, const float (&s)[N], float (&p)[N])
{
    float mt = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    if constexpr (N == 8) mt = fmaxf(mt, fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
    if (__any(mt > st.m)) {          // (the running maximum settles after a few tiles)
        float mn = fmaxf(st.m, mt);
        mn = fmaxf(mn, __shfl_xor(mn, 16, 64));
        mn = fmaxf(mn, __shfl_xor(mn, 32, 64));
        const float ms = mn == -INFINITY ? 0.f : mn;
        const float a = __builtin_amdgcn_exp2f(st.m - ms);
        st.l *= a;
        st.m = mn;
        const int g4 = (threadIdx.x & 48) >> 2;
        float f[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = __shfl(a, g4 + i, 64);        // factor of column 4g+i
#pragma unroll
        for (int d = 0; d < 8; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                st.o[d][i] *= f[i];
                if constexpr (StreamState<G>::kThird) st.o3[d][i] *= f[i];
            }
    }
    const float ms = st.m == -INFINITY ? 0.f : st.m;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        p[i] = __builtin_amdgcn_exp2f(s[i] - ms);
        st.l += p[i];
    }
}

__device__ __forceinline__ s16x4 upper_halves(const float (&x)[4])
{
    u32x2 w;
    w.x = __builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07060302u);
    w.y = __builtin_amdgcn_perm(__float_as_uint(x[3]), __float_as_uint(x[2]), 0x07060302u);
    return __builtin_bit_cast(s16x4, w);
}

// The parts of a probability above zero are at least 2^-126 (or the probability itself, if that is less): a part of zero
// times an infinite value would be NaN.  Where a part was less, this adds at most 2^-126 of a value: less than the
// rounding of the products for any probability above 2^-100, and nothing beside the row of the largest for the others.
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u16x4 part_floor(const float (&p)[4])
{
    const u16x4 tiny = {0x0080, 0x0080, 0x0080, 0x0080};        // (bf16 values of one sign compare like whole numbers)
    return __builtin_elementwise_min(__builtin_bit_cast(u16x4, upper_halves(p)), tiny);
}
__device__ __forceinline__ s16x4 raised(s16x4 part, u16x4 floor)
{
    return __builtin_bit_cast(s16x4, __builtin_elementwise_max(__builtin_bit_cast(u16x4, part), floor));
}

template <int G>
__device__ __forceinline__ void tile_values(StreamState<G>& st, const float (&p)[4], uint32_t v_addr, uint32_t mask1,
                                            uint32_t mask2)
{
    // this lane's part of p: p itself, what truncation to bf16 leaves, or what it leaves of that
    float x[4], y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = p[i] - __uint_as_float(__float_as_uint(p[i]) & mask1);
        if constexpr (StreamState<G>::kThird) {
            const float r = p[i] - __uint_as_float(__float_as_uint(p[i]) & 0xffff0000u);
            y[i] = r - __uint_as_float(__float_as_uint(r) & 0xffff0000u);
        } else {
            x[i] = x[i] - __uint_as_float(__float_as_uint(x[i]) & mask2);
        }
    }
    const u16x4 floor = part_floor(p);
    const s16x4 a = raised(upper_halves(x), floor);
    s16x4 v[8];
    const uint32_t a0 = v_addr, a1 = v_addr ^ 32u, a2 = v_addr ^ 64u, a3 = v_addr ^ 96u, a4 = v_addr ^ 128u,
                   a5 = v_addr ^ 160u, a6 = v_addr ^ 192u, a7 = v_addr ^ 224u;
    asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %9\n\tds_read_b64_tr_b16 %2, %10\n\t"
                 "ds_read_b64_tr_b16 %3, %11\n\tds_read_b64_tr_b16 %4, %12\n\tds_read_b64_tr_b16 %5, %13\n\t"
                 "ds_read_b64_tr_b16 %6, %14\n\tds_read_b64_tr_b16 %7, %15\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                 : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(a4), "v"(a5), "v"(a6), "v"(a7)
                 : "memory");
#pragma unroll
    for (int d = 0; d < 8; ++d) st.o[d] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, v[d], st.o[d], 0, 0, 0);
    if constexpr (StreamState<G>::kThird) {
        const s16x4 b = raised(upper_halves(y), floor);
#pragma unroll
        for (int d = 0; d < 8; ++d) st.o3[d] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(b, v[d], st.o3[d], 0, 0, 0);
    }
}

// Logits of rows 4g .. 4g+3 of a tile, stored row after row.
template <int G>
__device__ __forceinline__ void lds_read_scores(uint32_t a, float (&s)[4])
{
    asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:%5\n\tds_read_b32 %2, %4 offset:%6\n\t"
                 "ds_read_b32 %3, %4 offset:%7\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(s[0]), "=&v"(s[1]), "=&v"(s[2]), "=&v"(s[3])
                 : "v"(a), "n"(4 * G), "n"(8 * G), "n"(12 * G)
                 : "memory");
}

// Rows [w0, w1) of a source through one wave.  `ring`: LDS byte offset of the wave's ring; `strips`: of its two
// strips of row numbers.  kScored: the logits are ready-made; they take the place of the key rows in the ring.  (Fetched
// into registers when their tile was due, they made every tile a trip to memory of its own: one level of 4096 centroids,
// 64 / 256 units of 4 heads, whole step: 127.5 / 226.9 -> 122.5 / 205.0 us.)
// The first strip is on its way or there already (early_strip, take_guest_strip); `started` runs once it is in place, and
// may ask for one more strip.
template <int G, bool kScored, bool kListed, typename Started>
__device__ __forceinline__ void stream_tiles(StreamState<G>& st, const RowSource& S, const ValuePassParams& p, int u, int w0,
                                             int w1, uint32_t ring, uint32_t strips, Started started)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int head = c % G;                                       // (columns beyond the last part repeat a head)
    const int part = c / G;
    const uint32_t mask1 = part >= 1 ? 0xffff0000u : 0u, mask2 = part >= 2 ? 0xffff0000u : 0u;
    const unsigned char* Kb = reinterpret_cast<const unsigned char*>(S.K) + (long long)u * S.unit_rows * 256;
    const unsigned char* Vb = reinterpret_cast<const unsigned char*>(S.V) + (long long)u * S.unit_rows * 256;
    const int32_t* rows = kListed ? S.rows + (long long)u * S.rows_stride : nullptr;
    const float* scores = kScored ? S.scores + (long long)u * S.rows_stride * G : nullptr;

    // B operand: this column's query, dims [32 ks + 8 g, +8)
    bf16x8 q[4];
    if constexpr (!kScored) {
        const uint4* qp = reinterpret_cast<const uint4*>(p.q + ((long long)u * G + head) * kHeadDim);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) q[ks] = __builtin_bit_cast(bf16x8, qp[4 * ks + g]);
    }
    // LDS layout of a piece: row r at 256 r, its 16-byte chunk j at position j ^ r (conflict-free reads).
    // loads: instruction i covers rows 4i .. 4i+3, lane = 16 (row - 4i) + position
    const uint32_t chunk = (uint32_t)((c ^ g) * 16);              // ^ 64 i: byte offset of the chunk this lane loads
    const uint32_t k_addr = ring + (uint32_t)(c * 256 + ((g ^ c) & 3) * 16 + (c >> 2) * 64);      // ^ 64 ks
    const int vr = 4 * g + (c >> 2);
    const uint32_t v_addr = ring + (uint32_t)(vr * 256 + ((((c & 3) >> 1) ^ vr) & 1) * 16 + (c & 1) * 8 + (vr >> 1) * 32);   // ^ 32 d
    const int n_tiles = (w1 - w0 + kTile - 1) / kTile;
    constexpr int kBehind = kScored ? kScores : kPiece, kSlot = kBehind + kPiece;      // the ring: two slots, values behind keys or logits

    auto load_strip = [&](int s) {          // row numbers [w0 + 64 s, +64), clamped to the last row
        if constexpr (kListed) {
            int j = w0 + s * kStrip + lane;
            j = j < w1 ? j : w1 - 1;
            load_to_lds<4, false>(rows + j, strips + (uint32_t)((s & 1) * 4 * kStrip));
        }
    };
    long long off[4];                        // byte offsets of the rows this lane loads for a tile
    auto tile_rows = [&](int t) {
        int r[4];
        if constexpr (kListed) lds_read_rows(strips + (uint32_t)((((t >> 2) & 1) * kStrip + (t & 3) * kTile + g) * 4), r);
        if constexpr (kListed)
            if (t == n_tiles - 1) {          // (past the share's end a strip holds anything: the tile's first row instead)
                const int first = __builtin_amdgcn_readfirstlane(r[0]);
#pragma unroll
                for (int i = 0; i < 4; ++i) r[i] = w0 + t * kTile + 4 * i + g < w1 ? r[i] : first;
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (!kListed) r[i] = min(w0 + t * kTile + 4 * i + g, w1 - 1);
            off[i] = (long long)r[i] * 256 + (chunk ^ (uint32_t)(64 * i));
        }
    };
    constexpr int kKeyLoads = kScored ? (kTile * G + 63) / 64 : 4;       // instructions of load_keys
    auto load_keys = [&](int t) {
        if constexpr (kScored) {
#pragma unroll
            for (int i = 0; i < kKeyLoads; ++i) {
                const int x = min((w0 + t * kTile) * G + 64 * i + lane, w1 * G - 1);
                load_to_lds<4, false>(scores + x, ring + (uint32_t)((t & 1) * kSlot + i * 256));
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) load_to_lds<16, true>(Kb + off[i], ring + (uint32_t)((t & 1) * kSlot + i * 1024));
        }
    };
    auto load_values = [&](int t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) load_to_lds<16, true>(Vb + off[i], ring + (uint32_t)((t & 1) * kSlot + kBehind + i * 1024));
    };

    // The value rows of tile t past the end of the wave's share (repeats of its last row) are zeroed: their probability is
    // zero, and so is then their product whatever that row holds.
    auto clear_past_end = [&](int t, uint32_t piece) {
        const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (w0 + t * kTile + 4 * i + g >= w1)
                *reinterpret_cast<__attribute__((address_space(3))) u32x4*>((uintptr_t)(piece + (uint32_t)((4 * i + g) * 256 + c * 16))) = zero;
    };

    // In program order the loads of a wave are K0 V0 K1 V1 K2 V2 ..., four instructions a piece (logits in the place of keys:
    // one or two), and a strip of row numbers now and then.  Loads return in order, so "at most as many outstanding as the
    // pieces behind it have" in front of a piece's use means that it has arrived, and that every older strip has.  A
    // piece's slot is loaded again only after the LDS reads of the piece have returned.  Nothing is asked for past the end:
    // a share is often a single tile, and rows no one uses made its end wait for a second trip to memory (dense calls over
    // up to 8192 rows of 8 units, 4 heads: 12.5-15.1 -> 11.9-13.8 us).
    const bool single = n_tiles == 1;
    if constexpr (kListed) wait_vm<0>();
    tile_rows(0);
    if (n_tiles > kStrip / kTile) load_strip(1);
    load_keys(0);
    load_values(0);
    started();
    if (!single) {
        tile_rows(1);
        load_keys(1);
        load_values(1);
    }
    // kAhead: how many tiles follow (two: two or more)
    auto tile = [&](int t, auto ahead) {
        constexpr int kAhead = decltype(ahead)::value;
        const uint32_t half = (uint32_t)((t & 1) * kSlot);
        float s[4];
        wait_vm<kAhead == 0 ? 4 : 8 + kKeyLoads>();
        if constexpr (kScored) {
            lds_read_scores<G>(ring + half + (uint32_t)((4 * g * G + head) * 4), s);
            if constexpr (kAhead == 2) {
                tile_rows(t + 2);
                load_keys(t + 2);
            }
        } else {
            bf16x8 k[4];
            const uint32_t a0 = k_addr + half, a1 = (k_addr ^ 64u) + half, a2 = (k_addr ^ 128u) + half, a3 = (k_addr ^ 192u) + half;
            asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3])
                         : "v"(a0), "v"(a1), "v"(a2), "v"(a3)
                         : "memory");
            if constexpr (kAhead == 2) {
                tile_rows(t + 2);
                load_keys(t + 2);
            }
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[ks], q[ks], acc, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = acc[i] * p.scale_log2e;
        }
        if constexpr (kAhead == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = w0 + t * kTile + 4 * g + i < w1 ? s[i] : -INFINITY;
        }
        float pr[4];
        tile_softmax<G>(st, s, pr);
        wait_vm<kAhead == 2 ? 4 + 2 * kKeyLoads : kAhead * (4 + kKeyLoads)>();
        if constexpr (kAhead == 0) clear_past_end(t, ring + half + kBehind);
        tile_values<G>(st, pr, v_addr + half + kBehind, mask1, mask2);
        if constexpr (kAhead == 2) {
            load_values(t + 2);
            // the row numbers of tile t + 2, the last of its strip, have just been read: its slot takes the strip after next
            if constexpr (kListed)
                if ((t & 3) == 1 && ((t >> 2) + 2) * (kStrip / kTile) < n_tiles) load_strip((t >> 2) + 2);
        }
    };
    int t = 0;
    for (; t + 2 < n_tiles; ++t) tile(t, std::integral_constant<int, 2>{});
    if (!single) tile(t++, std::integral_constant<int, 1>{});
    tile(t, std::integral_constant<int, 0>{});
}

// The arguments span eight cache lines of a segment no one has read yet: one request for each of them, together.
__device__ __forceinline__ void touch_arguments(const ValuePassParams& p)
{
    static_assert(sizeof(ValuePassParams) <= 512 && sizeof(RowSource) == 120, "");
    asm volatile("" ::"s"(p.q), "s"(p.src[0].scores), "s"(p.src[0].guest), "s"(p.src[1].count_dev), "s"(p.src[1].guest),
                 "s"(p.src[2].count_max), "s"(p.src[2].guest), "s"(p.src[3].scores));
}

// What a workgroup works on: its unit, chunk and source, the rows [begin, end) of the chunk and [w0, w1) of this wave, and of
// the guest source (src[0], which rides along) the rows [g0, g1) and [a, b).
struct StreamShare {
    int u, chunk, source, begin, end, w0, w1, g0, g1, a, b;
};
// A launch over a short selection is a chain of trips to memory: arguments, counts, row numbers, rows, and the guest's row
// numbers and rows.  Each step is asked for as early as it can be (one level of 64 clusters, 1 unit: step 16.9 -> 16.4 us; 8 units x
// 4096 keys 28.6 -> 27.8; 32 units x 4096, 5 heads 42.0 -> 41.1).  The wave's first row numbers do not wait for the count: `early(source, unit, first position)` asks for them, and what lies past the end
// is never used as an address.
template <int kWaves, typename Early>
__device__ __forceinline__ StreamShare stream_share(const ValuePassParams& p, Early early)
{
    StreamShare r;
    r.chunk = blockIdx.x / p.n_units;
    const int u = r.u = blockIdx.x - r.chunk * p.n_units;
    r.source = 0;
#pragma unroll
    for (int i = 1; i < kMaxSources; ++i)
        if (i < p.n_sources && r.chunk >= p.src[i].chunk0) r.source = i;
    const RowSource& S = p.src[r.source];
    const RowSource& T = p.src[0];
    const int wave = threadIdx.x >> 6;
    r.begin = S.row0 + (r.chunk - S.chunk0) * S.chunk_rows;
    const int wave_rows = ((S.chunk_rows / kWaves) + kTile - 1) / kTile * kTile;
    r.w0 = r.begin + wave * wave_rows;
    // (the source's fields in one trip, the counts in one more)
    asm volatile("" ::"s"(S.rows), "s"(S.rows_stride), "s"(S.count_dev), "s"(S.count_max), "s"(S.scores), "s"(S.n_chunks), "s"(S.guest),
                 "s"(T.count_dev), "s"(T.count_max), "s"(S.K), "s"(S.V), "s"(S.unit_rows));
    typedef const __attribute__((address_space(4))) int32_t constant_int;
    int counted = 0, guests = 0;
    if (S.count_dev) counted = ((constant_int*)S.count_dev)[u];
    if (S.guest && T.count_dev) guests = ((constant_int*)T.count_dev)[u];
    if (S.rows) early(S, u, r.w0);
    int count = S.row0 + S.count_max;
    if (S.count_dev) count = counted < count ? counted : count;
    r.end = (r.begin + S.chunk_rows < count) ? r.begin + S.chunk_rows : count;
    r.g0 = r.g1 = 0;
    if (S.guest) {
        int nt = T.count_max;
        if (T.count_dev) nt = guests < nt ? guests : nt;
        const long long k = r.chunk - S.chunk0;
        r.g0 = (int)(nt * k / S.n_chunks);
        r.g1 = (int)(nt * (k + 1) / S.n_chunks);
    }
    r.w1 = (r.w0 + wave_rows < r.end) ? r.w0 + wave_rows : r.end;
    const int per = (((r.g1 - r.g0) + kWaves - 1) / kWaves + 15) & ~15;
    r.a = r.g0 + wave * per;
    r.b = (r.a + per < r.g1) ? r.a + per : r.g1;
    return r;
}
// The row numbers of 64 list positions from `first` to LDS, inside the unit's list.
__device__ __forceinline__ void fetch_strip(const int32_t* list, const RowSource& S, int u, int first, uint32_t to)
{
    const long long j = min((long long)first + (threadIdx.x & 63), S.rows_stride - 1);
    load_to_lds<4, false>(list + (long long)u * S.rows_stride + j, to);
}
// The guest source's first strip, fetched beside the main source's rows, takes the place of the first strip.
__device__ __forceinline__ void take_guest_strip(uint32_t from, uint32_t strips)
{
    wait_vm<0>();
    const uint32_t at = (threadIdx.x & 63) * 4;
    int row;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)\n\tds_write_b32 %2, %0\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(row) : "v"(from + at), "v"(strips + at) : "memory");
}
template <int G>
__device__ __forceinline__ void clear_state(StreamState<G>& st)
{
    st.m = -INFINITY;
    st.l = 0.f;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        st.o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (StreamState<G>::kThird) st.o3[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// The waves' sums become the workgroup's partial result; `sm`: LDS of the workgroup, whose waves may still be reading it.
template <int G, int kWaves>
__device__ __forceinline__ void combine_waves(const StreamState<G>& st, float* sm, float* part)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 4, c = lane & 15;
    float l = st.l;
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    __syncthreads();                         // (every wave is done with its ring)
    float* sm_m = sm;                        // [kWaves][16]
    float* sm_l = sm + 16 * kWaves;
    constexpr int kCols = StreamState<G>::kThird ? 16 + 8 : 16;
    float* sm_o = sm + 32 * kWaves;          // [kWaves][kCols][kRow]
    constexpr int kRow = 132;                // (the four rows a store instruction has are four apart: at 128 they would meet in one bank)
    if (lane < 16) {
        sm_m[wave * 16 + lane] = st.m;
        sm_l[wave * 16 + lane] = l;
    }
#pragma unroll
    for (int d = 0; d < 8; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sm_o[(wave * kCols + 4 * g + i) * kRow + 16 * d + c] = st.o[d][i];
            if constexpr (StreamState<G>::kThird)
                if (g < 2) sm_o[(wave * kCols + 16 + 4 * g + i) * kRow + 16 * d + c] = st.o3[d][i];
        }
    __syncthreads();
    for (int o = tid; o < G * 128; o += 64 * kWaves) {
        const int h = o >> 7, d = o & 127;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) M = fmaxf(M, sm_m[w * 16 + h]);
        const float Ms = M == -INFINITY ? 0.f : M;
        float a = 0.f, L = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float f = __builtin_amdgcn_exp2f(sm_m[w * 16 + h] - Ms);
            L = fmaf(sm_l[w * 16 + h], f, L);
            float x = sm_o[(w * kCols + h) * kRow + d];
            x += sm_o[(w * kCols + G + h) * kRow + d];
            x += sm_o[(w * kCols + (StreamState<G>::kThird ? 16 : 2 * G) + h) * kRow + d];
            a = fmaf(x, f, a);
        }
        float* ph = part + h * kPartStride;
        ph[4 + d] = a;
        if (d == 0) {
            ph[0] = M;
            ph[1] = L;
        }
    }
}

}  // namespace
}  // namespace mp
