// Centroid scoring and budgeted cluster selection for gfx950 (Eq. 1, Sec. 3.1; two levels: Sec. 3.4).
//
// One launch per decode step, one workgroup of 512 threads per unit; the coarse level and the fine
// level run back to back in the same workgroup.  The launch moves a few per cent of the step's
// bytes and nothing can overlap it (the value pass needs its result), so what counts is the length
// of the chain a wave executes: per level one trip to memory for the centroid rows, all requested at
// once, then a handful of short phases between workgroup barriers.  Two measured facts shape it:
//   * one compute unit pulls only about 20 GB/s out of a cold HBM (the chip's bandwidth is the sum
//     over its 256 units), so the 64-128 KiB of centroid rows per level are the largest single cost;
//   * with two waves per SIMD a wave issues one instruction in 5 cycles, a dependent one 8 cycles after its
//     predecessor (fp32 and fp64 alike; DPP 12, permlane swap 24, LDS read 67, fp64 division 70; a barrier 15;
//     code that runs for the first time is no slower), so the chain is kept short: the products run on the
//     fp64 matrix pipe and everything about an entry stays in the registers the product leaves it in (the
//     register path below).  (More waves would shorten the per-entry part and lengthen what every wave
//     does for itself: 512 threads is where the two balance for levels of 256-512 entries.)
//
// Logits l[h,i] = scale * q_h . Kc_i are accumulated in fp64 (products of bf16 numbers are exact,
// so the sum carries ~1e-16 relative error and the ranking agrees with an fp64 reference except on
// ties far below any tolerance) with v_mfma_f64_4x4x4 (four independent 4x4x4 blocks per
// instruction: 16 entries x 4 heads per wave and round).  The score of an entry is
// sum_h e^{l[h,i] - LSE_h}, G times Eq. 1 averaged over the query heads of the group; it is compared
// in the linear domain (same order as its logarithm, the rank key the getters report).  Selection =
// "take clusters in descending score order (ties: lower id) while the running token count stays
// within the budget, stop at the first that does not fit"; token counts are positive, so this is a
// threshold on (score, id): a 256-bucket histogram over the leading bits of the score and a direct
// comparison among the entries of the boundary bucket (where that bucket is crowded the register path
// divides it by up to two more digits; a most-significant-digit radix search takes over behind both).
//
// A level of at most lds_cap entries takes the register path (fast_level): its per-entry values live in
// registers, the candidate list and the compact list of selected clusters in LDS, and its barriers wait for LDS
// only.  Any other level works on arrays in a global scratch area, one entry per thread at a time (score_level).
//
// Shadow workgroups: with spare compute units (2 U <= units of the chip, U a multiple of eight: the
// blocks of a launch go round the eight L2 slices), a second workgroup per unit, placed on the same
// L2 slice, runs the same code without storing anything and asks for the centroid rows in the
// opposite order, so that each of the two finds part of its rows already in the shared L2.  It never
// communicates with the first.
//
// Helpers: where the units' fine clusters are few enough (score_helpers in mp_plan.h), further workgroups work out the
// logits of ALL fine clusters of a unit, and their exponentials, while its own workgroup is busy with the coarse level
// (early_logits).  They hand them over in global memory, past the L2 slices, which not all workgroups share: stored and loaded at
// device scope, and each helper counts itself in once its stores have arrived.  The unit's workgroup looks at the count when
// its candidates are known: if all helpers are done it loads 64 bytes a candidate (four heads) instead of the 256-byte row, its product
// and its exponentials, else it works the level out for itself -- it does not wait for workgroups that may not have
// started, so no order of dispatch is relied on, and the bits are the same either way.  Fine level of 256 candidates, 4 heads, up to the
// exponentials 11.7k -> 6.7k cycles, of 390, 8 heads 24.7k -> 11.1k; whole step, 8 units of 1024 clusters 27.4 -> 25.4 us, 24 of
// 1563 with 8 heads 47.3 -> 41.3.  In place of the shadow workgroup there.
//
// Outputs for the value pass: the flat list of stored rows of the selected clusters' keys, and one
// "centroid term" entry (value-centroid row + ready-made logits) per cluster that stays behind at
// either level (unpromising coarse clusters, unselected fine candidates).
#include <type_traits>

#include "mp_device.h"
#include "mp_internal.h"

namespace mp {

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kInFlight = 4;                          // rounds (16 entries per wave) whose centroid rows are requested ahead
constexpr int kHistBits = 8;                          // first (and normally only) digit of the selection
constexpr int kHistBuckets = 1 << kHistBits;
constexpr int kListCap = 64;                          // boundary-bucket entries ordered by direct comparison
static_assert(kThreads == 512, "a thread carries one element per head group of the 512-element query operand");
static_assert(kWaves <= 16, "the (head, wave) lane layout below uses rows of 16 lanes");
constexpr int kKeep = 2;                              // chunks of kThreads entries whose e^{l - M} stay in registers

// Order-preserving 64-bit image of a rank key r, ascending = descending r.
__device__ __forceinline__ uint64_t descending_key(double r)
{
    uint64_t b = (uint64_t)__double_as_longlong(r);
    b = (b >> 63) ? ~b : (b | 0x8000000000000000ull);   // ascending in r
    return ~b;                                           // ascending key = descending r
}

struct Scratch {
    unsigned long long hist[3][256];  // radix digit histograms: entry count << 40 | token count
    unsigned long long hkey[3][256];  // a key that fell into each bucket (THE key where the bucket holds one entry)
    unsigned long long rk_min[kWaves], rk_max[kWaves];  // per wave: smallest / largest key that takes part
    uint32_t rk_wt[kWaves], rk_cn[kWaves];              // ... their token total and their number
    uint32_t wsum[2][kWaves][2];      // per-wave totals of the two-value scan, double-buffered
    double wm[kWaves][8];             // per wave and head: largest logit of an entry that takes part
    double ws[kWaves][8];             // per wave and head: sum of N e^{l - M_h}
    double bm[8], bs[8];              // what stayed behind at the coarse level, per head: shift and sum of N e^{l - shift}
    double bw[kWaves][8];             // ... the same sum by wave (register path: bs is its column sums)
    uint32_t far[2];                  // register path, per level: some logit needs a shift
    uint32_t tiny;                    // register path: some score left the range of a double
    uint32_t early;                   // the helpers' logits are there
    // extremes of the keys, token total, "some score too small" flag and boundary-list length of the
    // level in progress, maintained with LDS atomics
    unsigned long long key_min, key_max;
    uint32_t key_total, key_tiny, bl_count;
    uint32_t ahead[kListCap];         // register path, per entry of the boundary list: tokens of the entries before it
};

struct Arrays {
    double* lg;            // [G][lg_stride]
    long long lg_stride;
    uint64_t* keys;
    uint32_t* wts;
    int32_t* ids;          // candidate fine ids (fine level of two)
    int32_t* aux;          // fine: first stored row; coarse: first child
    int32_t* aux2;         // coarse: end of children; fine: offset of the cluster's rows in the row list
    uint8_t* flags;
};

// Barrier between phases.  With the working arrays in LDS nothing written to global memory is read
// back inside the kernel, so only LDS traffic has to be ordered and outstanding global stores may
// stay in flight.
template <bool kLds>
__device__ __forceinline__ void phase_sync()
{
    if constexpr (kLds) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    } else {
        __syncthreads();
    }
}

// Inclusive prefix sum over lanes 0..7 (the same DPP row; what lies above them is of no interest).
__device__ __forceinline__ uint32_t eight_incl_scan_u32(uint32_t v)
{
    static_assert(kWaves == 8, "one lane per wave");
    v += dpp_u32_or0<0x111, 0xf>(v);
    v += dpp_u32_or0<0x112, 0xf>(v);
    v += dpp_u32_or0<0x114, 0xf>(v);
    return v;
}
// Exclusive prefix sums of two values per thread over one chunk of kThreads threads, with running
// totals carried in registers (every thread adds the same chunk totals, so they stay uniform).
// One barrier per call: the per-wave totals are double-buffered by the parity of `calls`; after the
// barrier the first 16 lanes of every wave scan them.
struct ScanState {
    uint32_t carry_a = 0, carry_b = 0, calls = 0;
};
template <bool kLds>
__device__ __forceinline__ void chunk_excl_scan2(uint32_t a, uint32_t b, Scratch& s, ScanState& st, uint32_t& ex_a,
                                                 uint32_t& ex_b)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t ia = wave_incl_scan_u32(a), ib = wave_incl_scan_u32(b);
    const int par = st.calls & 1;
    ++st.calls;
    if (lane == 63) {
        s.wsum[par][wave][0] = ia;
        s.wsum[par][wave][1] = ib;
    }
    phase_sync<kLds>();
    const uint32_t wa = lane < kWaves ? s.wsum[par][lane][0] : 0u, wb = lane < kWaves ? s.wsum[par][lane][1] : 0u;
    const uint32_t sa = eight_incl_scan_u32(wa), sb = eight_incl_scan_u32(wb);
    const int w = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t off_a = (uint32_t)__builtin_amdgcn_readlane((int)(sa - wa), w);
    const uint32_t off_b = (uint32_t)__builtin_amdgcn_readlane((int)(sb - wb), w);
    const uint32_t tot_a = (uint32_t)__builtin_amdgcn_readlane((int)sa, kWaves - 1);
    const uint32_t tot_b = (uint32_t)__builtin_amdgcn_readlane((int)sb, kWaves - 1);
    ex_a = st.carry_a + off_a + ia - a;
    ex_b = st.carry_b + off_b + ib - b;
    st.carry_a += tot_a;
    st.carry_b += tot_b;
}

template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, Op op)
{
    auto moved = [](T x, auto ctrl) {
        constexpr int kCtrl = decltype(ctrl)::value;
        if constexpr (sizeof(T) == 4) {
            return (T)__builtin_amdgcn_mov_dpp((int)x, kCtrl, 0xf, 0xf, true);
        } else {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, kCtrl, 0xf, 0xf, true);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), kCtrl, 0xf, 0xf, true);
            return (T)(((uint64_t)hi << 32) | lo);
        }
    };
    auto lane_value = [](T x, int src) {
        if constexpr (sizeof(T) == 4) {
            return (T)__builtin_amdgcn_readlane((int)x, src);
        } else {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, src);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), src);
            return (T)(((uint64_t)hi << 32) | lo);
        }
    };
    v = op(v, moved(v, std::integral_constant<int, kDppXor1>{}));
    v = op(v, moved(v, std::integral_constant<int, kDppXor2>{}));
    v = op(v, moved(v, std::integral_constant<int, kDppHalfMirror>{}));
    v = op(v, moved(v, std::integral_constant<int, kDppMirror>{}));
    return op(op(lane_value(v, 0), lane_value(v, 16)), op(lane_value(v, 32), lane_value(v, 48)));
}

// Weighted radix select.  keys[i] ascending = rank order, wts[i] > 0 for entries that take part
// (entries with wts == 0 are never selected).  Finds the key K* of the first entry (in (key, index)
// order) at which the running weight exceeds `budget`, the weight `acc` of all entries with key <
// K*, and how many entries carry exactly K*.  Returns false if everything fits.
//
// Digits are taken from key - min(key), starting at the top bit of max - min, so that the first
// digit already spreads the entries over the histogram instead of piling them onto a few LDS
// addresses.  One barrier per digit of up to 8 bits: the histogram (entry count and token count
// packed in one 64-bit LDS atomic) is scanned by every wave for itself, which leaves the chosen
// digit wave-uniform in registers.  Next to each bucket's counts sits the key of an entry that fell
// into it, so that the pass in which the boundary bucket is down to one entry ends the search
// without another sweep.  Three histogram buffers rotate: pass p fills buffer p%3 and
// clears buffer (p+1)%3, whose last readers (pass p-2) all finished before the barrier of pass p-1.
template <bool kLds>
__device__ __forceinline__ bool radix_select(const uint64_t* keys, const uint32_t* wts, int n, long long budget,
                                             Scratch& s, uint64_t& kstar, uint64_t& acc_out, uint32_t& ties_out)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr unsigned long long kWtMask = (1ull << 40) - 1;
    // token totals fit 31 bits
    const uint32_t bud = budget < 0 ? 0u : (budget > 0xffffffffll ? 0xffffffffu : (uint32_t)budget);
    {
        uint64_t kmin = ~0ull, kmax = 0;
        uint32_t wt = 0, cn = 0;
        for (int i = tid; i < n; i += kThreads) {
            const uint32_t w = wts[i];
            if (w == 0) continue;
            const uint64_t k = keys[i];
            kmin = k < kmin ? k : kmin;
            kmax = k > kmax ? k : kmax;
            wt += w;
            ++cn;
        }
        kmin = wave_reduce(kmin, [](uint64_t a, uint64_t b) { return a < b ? a : b; });
        kmax = wave_reduce(kmax, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
        wt = wave_reduce(wt, [](uint32_t a, uint32_t b) { return a + b; });
        cn = wave_reduce(cn, [](uint32_t a, uint32_t b) { return a + b; });
        if (lane == 0) {
            s.rk_min[wave] = kmin;
            s.rk_max[wave] = kmax;
            s.rk_wt[wave] = wt;
            s.rk_cn[wave] = cn;
        }
    }
    if (tid < 256) s.hist[0][tid] = 0;
    phase_sync<kLds>();
    uint64_t kmin = ~0ull, kmax = 0;
    uint32_t total = 0, cnt = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint64_t a = s.rk_min[w], b = s.rk_max[w];
        kmin = a < kmin ? a : kmin;
        kmax = b > kmax ? b : kmax;
        total += s.rk_wt[w];
        cnt += s.rk_cn[w];
    }
    if (total <= bud) return false;           // everything fits
    const uint64_t range = kmax - kmin;
    int hi = range ? 64 - __clzll((long long)range) : 0;   // number of low bits of key - kmin still undecided
    uint64_t prefix = 0;                                   // the decided bits of K* - kmin
    uint32_t acc = 0;
    for (int pass = 0; hi > 0; ++pass) {
        const int bits = hi < 8 ? hi : 8, shift = hi - bits;
        const uint32_t dmask = (1u << bits) - 1u;
        unsigned long long* H = s.hist[pass % 3];
        unsigned long long* HK = s.hkey[pass % 3];
        if (tid < 256) s.hist[(pass + 1) % 3][tid] = 0;
        for (int i = tid; i < n; i += kThreads) {
            const uint32_t w = wts[i];
            if (w == 0) continue;
            const uint64_t k = keys[i] - kmin;
            if (hi >= 64 || (k >> hi) == prefix) {
                const uint32_t b = (uint32_t)(k >> shift) & dmask;
                atomicAdd(&H[b], (1ull << 40) | w);
                HK[b] = keys[i];        // plain store: only read back where this entry is alone in its bucket
            }
        }
        phase_sync<kLds>();
        unsigned long long h4[4];
        uint32_t sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            h4[j] = H[4 * lane + j];
            sum += (uint32_t)(h4[j] & kWtMask);
        }
        const uint32_t incl = wave_incl_scan_u32(sum);
        // the bucket being split weighs more than what is left of the budget, so some lane crosses
        const unsigned long long mask = __ballot((unsigned long long)acc + incl > bud);
        const int first = mask ? __ffsll((long long)mask) - 1 : 63;
        uint32_t a = acc + incl - sum, d = 4 * lane, c = 0;
        bool done = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t wj = (uint32_t)(h4[j] & kWtMask);
            if (!done) {
                if ((unsigned long long)a + wj > bud) {
                    d = 4 * lane + j;
                    c = (uint32_t)(h4[j] >> 40);
                    done = true;
                } else {
                    a += wj;
                }
            }
        }
        acc = (uint32_t)__builtin_amdgcn_readlane((int)a, first);
        cnt = (uint32_t)__builtin_amdgcn_readlane((int)c, first);
        prefix = (prefix << bits) | (uint32_t)__builtin_amdgcn_readlane((int)d, first);
        hi = shift;
        if (cnt == 1 && hi > 0) {
            // a single entry carries the boundary: its full key is K*, and it left that key in the
            // bucket's slot (nobody else wrote there in this pass)
            kstar = HK[(uint32_t)prefix & dmask];
            acc_out = acc;
            ties_out = 1;
            return true;
        }
    }
    kstar = kmin + prefix;
    acc_out = acc;
    ties_out = cnt;
    return true;
}

// ------------------------------------------------------------------------------------------------
// Dynamic LDS behind the Scratch block: the query in matrix-operand order, the selection's
// histogram and boundary list, then the per-entry working arrays (cap = p.lds_cap entries each).
// ------------------------------------------------------------------------------------------------
struct Lds {
    double* qB;                 // [GH][32][16]: slice s, dim group k, head j (see query_operand_element)
    unsigned long long* hist;   // [kHistBuckets] entry count << 40 | token count
    unsigned long long* blist;  // [kListCap][2]: key, position << 32 | token count
    Arrays A;
};

__host__ __device__ constexpr size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

template <int G>
__device__ __forceinline__ Lds carve_lds(unsigned char* lds, int cap)
{
    constexpr int GH = (G + 3) / 4;
    Lds L;
    L.qB = reinterpret_cast<double*>(lds);
    L.hist = reinterpret_cast<unsigned long long*>(L.qB + GH * 512);
    L.blist = L.hist + kHistBuckets;
    L.A.lg = nullptr;            // (logits, row starts and flags of such a level stay in registers)
    L.A.lg_stride = 0;
    L.A.keys = reinterpret_cast<uint64_t*>(L.blist + 2 * kListCap);
    L.A.wts = reinterpret_cast<uint32_t*>(L.A.keys + cap);
    L.A.ids = reinterpret_cast<int32_t*>(L.A.wts + cap);
    L.A.aux2 = L.A.ids + cap;
    L.A.aux = nullptr;
    L.A.flags = nullptr;
    return L;
}

template <int G>
__device__ __forceinline__ Arrays global_arrays(const ScoreParams& p, int u)
{
    Arrays A;
    A.lg = p.lg + (long long)u * G * p.lg_stride;
    A.lg_stride = p.lg_stride;
    A.keys = reinterpret_cast<uint64_t*>(p.g_keys) + (long long)u * p.g_stride;
    A.wts = p.g_wts + (long long)u * p.g_stride;
    A.ids = p.cand + (long long)u * p.f_stride;       // the candidate list itself
    A.aux = p.g_aux + (long long)u * p.g_stride;
    A.aux2 = p.g_aux2 + (long long)u * p.g_stride;
    A.flags = p.g_flags + (long long)u * p.g_stride;
    return A;
}

// ------------------------------------------------------------------------------------------------
// The matrix product.
//
// v_mfma_f64_4x4x4 computes four independent blocks D_b[i][j] += sum_k A_b[i][k] * B_b[k][j] with
// (measured lane map) A_b[i][k] in lane 16k + 4b + i, B_b[k][j] in lane 16k + 4b + j and D_b[i][j]
// in lane 16i + 4b + j.  Here i = entry inside a block, j = head, k = one of four groups of 32
// dimensions: lane (k, e = 4b + i) holds, for entry e of the wave's 16, the dimensions
// {32c + 8k + r : c < 4, r < 8} (four 16-byte pieces of the row, so that one load instruction of the
// wave covers 64 contiguous bytes of 16 rows), and 32 instructions, one per (c, r), add up the whole
// product.  The B operand (the query, the same for every block) is read from LDS: element x of qB,
// x = (hg * 32 + 8c + r) * 16 + 4k + j, is dimension 32c + 8k + r of head 4 hg + j.
// After the product lane (i, b, j) owns the logit of entry 4b + i and head j.
// ------------------------------------------------------------------------------------------------
// Thread x carries element x of every head group, as bf16 until it is needed: loaded without a branch (a head past the last
// reads the last one's and counts as zero later), so that nothing waits for it before the rows have been asked for.
template <int G>
__device__ __forceinline__ uint16_t query_operand_element(const uint16_t* q, int u, int hg, int x)
{
    const int s = x >> 4, k = (x >> 2) & 3, h = min(4 * hg + (x & 3), G - 1), d = 32 * (s >> 3) + 8 * k + (s & 7);
    return q[((long long)u * G + h) * kHeadDim + d];
}

template <int G>
__device__ __forceinline__ double query_operand(uint16_t v, int hg, int x)
{
    return 4 * hg + (x & 3) < G ? (double)bf16_to_f32(v) : 0.0;
}

constexpr int kDppRowRor4 = 0x124, kDppRowRor8 = 0x128;
// The two halves of a pairwise exchange across rows of 16 lanes (kSpan = 16: rows 0/1 and 2/3; 32: the halves of
// the wave), as one vector instruction per 32 bits: op(first, second) is the same in all lanes concerned.
template <int kSpan>
__device__ __forceinline__ void exchange_u32(uint32_t v, uint32_t& first, uint32_t& second)
{
    const auto r = kSpan == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false)
                               : __builtin_amdgcn_permlane32_swap(v, v, false, false);
    first = r[0];
    second = r[1];
}
template <int kSpan, typename Op>
__device__ __forceinline__ double across_rows(double v, Op op)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    uint32_t l0, l1, h0, h1;
    exchange_u32<kSpan>((uint32_t)b, l0, l1);
    exchange_u32<kSpan>((uint32_t)(b >> 32), h0, h1);
    return op(__longlong_as_double((long long)(((unsigned long long)h0 << 32) | l0)),
              __longlong_as_double((long long)(((unsigned long long)h1 << 32) | l1)));
}
// Combination over the 16 lanes of a wave that are equal modulo 4 (matrix layout: the same head); every one of
// them receives the result.
template <typename Op>
__device__ __forceinline__ double same_head(double x, Op op)
{
    x = op(x, dpp_f64<kDppRowRor4>(x));
    x = op(x, dpp_f64<kDppRowRor8>(x));
    x = across_rows<16>(x, op);
    return across_rows<32>(x, op);
}
struct MaxOp { __device__ __forceinline__ double operator()(double a, double b) const { return fmax(a, b); } };
struct AddOp { __device__ __forceinline__ double operator()(double a, double b) const { return a + b; } };
// Sum over the wave; every lane receives it.
__device__ __forceinline__ uint32_t wave_total_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor1, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor2, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppRowRor4, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppRowRor8, 0xf, 0xf, true);
    uint32_t a, b;
    exchange_u32<16>(v, a, b);
    v = a + b;
    exchange_u32<32>(v, a, b);
    return a + b;
}
// The value lane t of each group of four holds.
template <int t>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, t * 0x55, 0xf, 0xf, true);
}
// Largest value over the 16 lanes of a wave that own the same head (lanes equal modulo 4).
__device__ __forceinline__ double max_same_head(double x) { return same_head(x, MaxOp{}); }
__device__ __forceinline__ double row_min_f64(double v)
{
    v = fmin(v, dpp_f64<kDppXor1>(v));
    v = fmin(v, dpp_f64<kDppXor2>(v));
    v = fmin(v, dpp_f64<kDppHalfMirror>(v));
    v = fmin(v, dpp_f64<kDppMirror>(v));
    return v;
}

// One value per head from a [kWaves][8] table of per-wave values: lane 16 hh + w of every wave takes
// the value of (wave w, head 4 hg + hh), the row is combined, `post` (head group, head, combined value) is applied
// -- once per head group, the heads side by side in the lanes -- and every lane receives the G results.
template <int G, typename RowOp, typename Post>
__device__ __forceinline__ void combine_waves(const double (&tab)[kWaves][8], double neutral, RowOp row_op, Post post,
                                              double (&out)[G])
{
    constexpr int GH = (G + 3) / 4;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int hg = 0; hg < GH; ++hg) {
        const int h = 4 * hg + (lane >> 4), w = lane & 15;
        const int hc = h < G ? h : G - 1;
        const double v = post(hg, hc, row_op((h < G && w < kWaves) ? tab[w][h] : neutral));
#pragma unroll
        for (int hh = 0; hh < 4; ++hh)
            if (4 * hg + hh < G) out[4 * hg + hh] = readlane_f64(v, 16 * hh);
    }
}

// The value itself, but the compiler can neither move its evaluation out of the branch it stands in nor
// evaluate it ahead of time (used to keep rarely needed logarithms out of the common path).
__device__ __forceinline__ double not_hoisted(double v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// One centroid-term entry (Eq. 2): the row of the value centroid and log2( N_i e^{l[h,i]} ) per head.
template <int G>
__device__ __forceinline__ void emit_term(const ScoreParams& p, const Arrays& A, int u, int i, int row, uint32_t slot)
{
    const long long o = (long long)u * p.mp_stride + slot;
    p.mp_rows[o] = row;
    const float lgN = __builtin_amdgcn_logf((float)A.wts[i]);
#pragma unroll
    for (int h = 0; h < G; ++h) p.mp_scores[o * G + h] = (float)(A.lg[h * A.lg_stride + i] * 1.4426950408889634) + lgN;
}

// The bucket of a histogram (entry count << 40 | token count each) in which the running token count, `before` to start
// with, passes the budget; what lies before that bucket and how many entries it holds.  Every wave scans the histogram
// for itself, kHistBuckets / 64 buckets per lane.
struct Boundary {
    uint32_t before, entries, bucket;
};
__device__ __forceinline__ Boundary find_boundary(const unsigned long long* hist, uint32_t before, uint32_t budget)
{
    constexpr unsigned long long kWtMask = (1ull << 40) - 1;
    constexpr int BPL = kHistBuckets / 64;
    const int lane = threadIdx.x & 63;
    unsigned long long hb[BPL];
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < BPL; ++i) {
        hb[i] = hist[BPL * lane + i];
        sum += (uint32_t)(hb[i] & kWtMask);
    }
    const uint32_t incl = before + wave_incl_scan_u32(sum);
    const unsigned long long crossing = __ballot((unsigned long long)incl > budget);
    const int first = crossing ? __ffsll((long long)crossing) - 1 : 63;
    uint32_t a = incl - sum, d = BPL * lane, cn = 0;
    bool done = false;
#pragma unroll
    for (int i = 0; i < BPL; ++i) {
        const uint32_t wi = (uint32_t)(hb[i] & kWtMask);
        if (!done) {
            if ((unsigned long long)a + wi > budget) {
                d = BPL * lane + i;
                cn = (uint32_t)(hb[i] >> 40);
                done = true;
            } else {
                a += wi;
            }
        }
    }
    return Boundary{(uint32_t)__builtin_amdgcn_readlane((int)a, first), (uint32_t)__builtin_amdgcn_readlane((int)cn, first),
                    (uint32_t)__builtin_amdgcn_readlane((int)d, first)};
}

// The flat list of stored rows of the selected clusters, from (first stored row, count) and offset of each: one row of 16
// lanes per cluster, the next cluster's entry fetched early.
__device__ __forceinline__ void expand_rows(const ScoreParams& p, int u, const int2* sel_rc, const int32_t* sel_off, uint32_t n_sel)
{
    const int grp = threadIdx.x >> 4, sub = threadIdx.x & 15;
    int32_t* ro = p.rows + (long long)u * p.rows_stride;
    int32_t* so = p.row_slot ? p.row_slot + (long long)u * p.rows_stride : nullptr;   // compact slot of each row's cluster
    int2 rc_n = make_int2(0, 0);
    int off_n = 0;
    if ((uint32_t)grp < n_sel) {
        rc_n = sel_rc[grp];
        off_n = sel_off[grp];
    }
    for (uint32_t k = grp; k < n_sel; k += kThreads / 16) {
        const int2 rc = rc_n;
        const int off = off_n;
        const uint32_t kn = k + kThreads / 16;
        if (kn < n_sel) {
            rc_n = sel_rc[kn];
            off_n = sel_off[kn];
        }
        for (int i = sub; i < rc.y; i += 16) ro[off + i] = rc.x + i;
        if (so)
            for (int i = sub; i < rc.y; i += 16) so[off + i] = (int32_t)k;
    }
}
__device__ __forceinline__ void write_counters(const ScoreParams& p, int u, uint32_t total, uint32_t n_terms, int n_f, bool two)
{
    if (threadIdx.x != 0) return;
    p.n_rows[u] = (int32_t)total;
    p.n_mp[u] = (int32_t)n_terms;
    p.counters[4 * u + 0] = (int32_t)total + p.n_tail;
    p.counters[4 * u + 1] = n_f;
    if (!two) p.counters[4 * u + 2] = 0;
    p.counters[4 * u + 3] = (int32_t)n_terms;
}

// One level: logits, Eq. 1 normaliser, scores, budgeted selection.
// Entry x stands for cluster id (use_ids ? A.ids[x] : x).  `with_behind`: the normaliser also covers
// the coarse clusters that stayed behind (S.bm / S.bs).  `q_pending`: the query operand still has to go
// to LDS (first level of the launch; qv = this thread's element).  On return A holds logits, keys,
// member counts (0 = takes no part), row starts and flags, all published by a barrier.  Returns 1 if
// the keys are linear-domain scores, 0 if they are logarithmic rank keys (the rare case of scores
// below the range of a double).
// What a level keeps of its own entries after the selection: the shift per head, and for the first
// kKeep chunks of kThreads entries the member count and e^{l - shift} of this thread's entry.
template <int G>
struct LevelState {
    double M[G];
    double ek[kKeep][G];
    uint32_t wk[kKeep];
};

template <int G>
__device__ __forceinline__ int score_level(const ScoreParams& p, const Lds& L, const Arrays& A, Scratch& S, int u, int n,
                                           bool use_ids, bool coarse, long long budget, bool with_behind,
                                           bool q_pending, const uint16_t (&qv)[(G + 3) / 4],
                                           unsigned long long* key_out, uint8_t* flag_out, LevelState<G>& state)
{
    constexpr int GH = (G + 3) / 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double ninf = -INFINITY;
    const int row_off = coarse ? p.fcap : 0;
    const int32_t* Nu = p.N + (long long)u * p.tab_rows + row_off;
    const uint16_t* Kcu = p.Kc + ((long long)u * p.tab_rows + row_off) * kHeadDim;
    const int32_t* st = coarse ? p.cstart + (long long)u * p.cstart_stride : p.fstart + (long long)u * p.fstart_stride;
    const int chunks = (n + kThreads - 1) / kThreads;

    // ================= logits: matrix layout, 16 entries per wave and round =================
    {
        const int kA = lane >> 4, eA = lane & 15;                       // operand layout: dim group, entry
        const int jD = lane & 3, eD = ((lane >> 2) & 3) * 4 + (lane >> 4);   // result layout: head, entry
        const int bsel = kA * 4 + jD;                                   // this lane's slot in a slice of qB
        const int rounds = (n + 16 * kWaves - 1) / (16 * kWaves);
        uint4 raw[kInFlight][4];
        int cntD[kInFlight], auxD[kInFlight], aux2D[kInFlight];
        auto request = [&](int t, uint4 (&r)[4], int& cnt, int& a1, int& a2) {
            const int base = (t * kWaves + wave) * 16;
            const int xa = base + eA, xd = base + eD;
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = make_uint4(0, 0, 0, 0);
            cnt = a1 = a2 = 0;
            if (xa < n) {
                const int id = use_ids ? A.ids[xa] : xa;
                const uint4* kp = reinterpret_cast<const uint4*>(Kcu + (long long)id * kHeadDim) + kA;
#pragma unroll
                for (int c = 0; c < 4; ++c) r[c] = kp[4 * c];
            }
            if (xd < n) {
                const int id = use_ids ? A.ids[xd] : xd;
                cnt = Nu[id];
                a1 = st[id];
                if (coarse) a2 = st[id + 1];
            }
        };
#pragma unroll
        for (int t = 0; t < kInFlight; ++t) {
            if (t < rounds) request(t, raw[t], cntD[t], auxD[t], aux2D[t]);
            else {
#pragma unroll
                for (int c = 0; c < 4; ++c) raw[t][c] = make_uint4(0, 0, 0, 0);
                cntD[t] = auxD[t] = aux2D[t] = 0;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // while the rows travel: empty histogram and extremes for this level's selection (their last
        // readers passed a barrier long ago), and the query operand
        if (tid < kHistBuckets) L.hist[tid] = 0;
        if (tid == 0) {
            S.bl_count = 0;
            S.key_min = ~0ull;
            S.key_max = 0;
            S.key_total = 0;
            S.key_tiny = 0;
        }
        if (q_pending) {
#pragma unroll
            for (int hg = 0; hg < GH; ++hg) L.qB[tid + hg * kThreads] = query_operand<G>(qv[hg], hg, tid);
            phase_sync<true>();
        }

        double mx[GH];
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) mx[hg] = ninf;
#pragma unroll 1
        for (int t0 = 0; t0 < rounds; t0 += kInFlight) {
#pragma unroll
            for (int j = 0; j < kInFlight; ++j) {
                const int t = t0 + j;
                if (t < rounds) {
                    double acc[GH];
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) acc[hg] = 0.0;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint32_t w4[4] = {raw[j][c].x, raw[j][c].y, raw[j][c].z, raw[j][c].w};
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const double a = (double)((e & 1) ? bf16hi_to_f32(w4[e >> 1]) : bf16lo_to_f32(w4[e >> 1]));
#pragma unroll
                            for (int hg = 0; hg < GH; ++hg)
                                acc[hg] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, L.qB[(hg * 32 + 8 * c + e) * 16 + bsel], acc[hg], 0, 0, 0);
                        }
                    }
                    const int xd = (t * kWaves + wave) * 16 + eD;
                    const bool part = xd < n && cntD[j] > 0;
                    if (xd < n && jD == 0) {
                        A.wts[xd] = part ? (uint32_t)cntD[j] : 0u;
                        A.aux[xd] = auxD[j];
                        if (coarse) A.aux2[xd] = aux2D[j];
                    }
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) {
                        const double l = acc[hg] * p.scale;
                        if (xd < n && 4 * hg + jD < G) {
                            A.lg[(4 * hg + jD) * A.lg_stride + xd] = l;
                            if (part) mx[hg] = fmax(mx[hg], l);
                        }
                    }
                    if (t + kInFlight < rounds) request(t + kInFlight, raw[j], cntD[j], auxD[j], aux2D[j]);
                }
            }
        }
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) {
            mx[hg] = max_same_head(mx[hg]);
            if (lane < 4 && 4 * hg + lane < G) S.wm[wave][4 * hg + lane] = mx[hg];
        }
    }
    __syncthreads();

    // ================= from here on thread tid owns entry tid (+ kThreads per further chunk) =================
    // shift of the level: the largest logit that takes part (and the shift of what stayed behind)
    double (&M)[G] = state.M;
    combine_waves<G>(S.wm, ninf, [](double v) { return row_max_f64(v); },
                     [&](int, int h, double v) { return (with_behind && S.bs[h] > 0.0) ? fmax(v, S.bm[h]) : v; }, M);
    // e^{l - M_h} of the own entries (kept in registers for the first kKeep chunks) and the sums of N e^{l - M_h}
    double (&ek)[kKeep][G] = state.ek;
    uint32_t (&wk)[kKeep] = state.wk;
    double sm[G];
#pragma unroll
    for (int h = 0; h < G; ++h) sm[h] = 0.0;
#pragma unroll
    for (int c = 0; c < kKeep; ++c) {
        wk[c] = 0;
#pragma unroll
        for (int h = 0; h < G; ++h) ek[c][h] = 0.0;
        const int i = tid + c * kThreads;
        if (i < n) wk[c] = A.wts[i];
        if (wk[c]) {
#pragma unroll
            for (int h = 0; h < G; ++h) {
                ek[c][h] = exp_shifted(A.lg[h * A.lg_stride + i] - M[h]);
                sm[h] += (double)wk[c] * ek[c][h];
            }
        }
    }
    for (int c = kKeep; c < chunks; ++c) {
        const int i = tid + c * kThreads;
        const uint32_t w = i < n ? A.wts[i] : 0u;
        if (w) {
#pragma unroll
            for (int h = 0; h < G; ++h) sm[h] += (double)w * exp_shifted(A.lg[h * A.lg_stride + i] - M[h]);
        }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {
        const double t = wave_sum_f64(sm[h]);
        if (lane == 0) S.ws[wave][h] = t;
    }
    __syncthreads();
    // 1 / sum_i N_i e^{l - M_h} per head (0 where nothing takes part)
    double inv[G];
    combine_waves<G>(S.ws, 0.0, [](double v) { return row_sum_f64(v); },
                     [&](int, int h, double v) {
                         if (with_behind && S.bs[h] > 0.0) {
                             // this row's head: its shift once more, from the table (cheaper than routing M here)
                             const int w = lane & 15;
                             const double m = fmax(row_max_f64(w < kWaves ? S.wm[w][h] : ninf), S.bm[h]);
                             v += S.bs[h] * exp_shifted(S.bm[h] - m);
                         }
                         return v > 0.0 ? 1.0 / v : 0.0;
                     }, inv);

    // ---- keys.  Linear domain: the complement of the bit pattern of sum_h e^{l - LSE_h} (ascending
    // key = descending score).  If a score leaves the range of a double, the whole level ranks by
    // log mean_h e^{l - LSE_h} worked out in the log domain instead (second trip; uniform). ----
    int linear = 1;
    constexpr double kLogGs[9] = {0.0, 0.0, 0.6931471805599453094, 1.0986122886681097821, 1.3862943611198906188,
                                  1.6094379124341002818, 1.7917594692280549573, 1.9459101090932196052, 2.0794415416798357477};
    constexpr double kLogG = kLogGs[G];
    for (;;) {
        double smin = INFINITY, smax = ninf;     // extremes of the score (linear) / of the rank key (log)
        uint32_t wsum = 0;
        bool tiny = false;
        auto one_key = [&](int i, uint32_t w, const double (&e)[G], bool kept) {
            uint64_t key = ~0ull;
            if (w) {
                double sc;
                if (linear) {
                    sc = 0.0;
#pragma unroll
                    for (int h = 0; h < G; ++h)
                        sc += (kept ? e[h] : exp_shifted(A.lg[h * A.lg_stride + i] - M[h])) * inv[h];
                    tiny |= !(sc >= 1e-280);
                    key = ~(uint64_t)__double_as_longlong(sc);
                } else {
                    double th[G], tm = ninf;
#pragma unroll
                    for (int h = 0; h < G; ++h) {
                        th[h] = A.lg[h * A.lg_stride + i] - (M[h] - log(not_hoisted(inv[h])));
                        tm = fmax(tm, th[h]);
                    }
                    double ss = 0.0;
#pragma unroll
                    for (int h = 0; h < G; ++h) ss += exp_shifted(th[h] - tm);
                    sc = tm - kLogG + log(ss);
                    key = descending_key(sc);
                }
                smin = fmin(smin, sc);
                smax = fmax(smax, sc);
                wsum += w;
            }
            if (i < n) {
                A.keys[i] = key;
                key_out[i] = key;
            }
        };
#pragma unroll
        for (int c = 0; c < kKeep; ++c)
            if (c < chunks) one_key(tid + c * kThreads, wk[c], ek[c], true);
        for (int c = kKeep; c < chunks; ++c) {
            const int i = tid + c * kThreads;
            one_key(i, i < n ? A.wts[i] : 0u, ek[0], false);
        }
        smin = row_min_f64(smin);
        smax = row_max_f64(smax);
        smin = fmin(fmin(readlane_f64(smin, 0), readlane_f64(smin, 16)), fmin(readlane_f64(smin, 32), readlane_f64(smin, 48)));
        smax = fmax(fmax(readlane_f64(smax, 0), readlane_f64(smax, 16)), fmax(readlane_f64(smax, 32), readlane_f64(smax, 48)));
        wsum = wave_reduce(wsum, [](uint32_t a, uint32_t b) { return a + b; });
        if (lane == 0 && wsum) {
            // the largest score carries the smallest key
            const uint64_t klo = linear ? ~(uint64_t)__double_as_longlong(smax) : descending_key(smax);
            const uint64_t khi = linear ? ~(uint64_t)__double_as_longlong(smin) : descending_key(smin);
            atomicMin(&S.key_min, (unsigned long long)klo);
            atomicMax(&S.key_max, (unsigned long long)khi);
            atomicAdd(&S.key_total, wsum);
        }
        if (__any(tiny) && lane == 0) atomicOr(&S.key_tiny, 1u);
        __syncthreads();
        if (!linear || !S.key_tiny) break;
        linear = 0;
        __syncthreads();       // everyone has seen the flag
        if (tid == 0) {
            S.key_min = ~0ull;
            S.key_max = 0;
            S.key_total = 0;
            S.key_tiny = 0;
        }
        __syncthreads();
    }

    // ---- budgeted selection ----
    const uint64_t kmin = S.key_min, kmax = S.key_max;
    const uint32_t total = S.key_total;
    const uint32_t bud = budget < 0 ? 0u : (budget > 0xffffffffll ? 0xffffffffu : (uint32_t)budget);
    if (total <= bud) {
        for (int c = 0; c < chunks; ++c) {
            const int i = tid + c * kThreads;
            if (i < n) {
                const uint8_t f = A.wts[i] ? 1 : 0;
                A.flags[i] = f;
                flag_out[i] = f;
            }
        }
    } else {
        const uint64_t range = kmax - kmin;
        const int hi = range ? 64 - __clzll((long long)range) : 0;
        const int bits = hi < kHistBits ? hi : kHistBits, shift = hi - bits;
        for (int c = 0; c < chunks; ++c) {
            const int i = tid + c * kThreads;
            const uint32_t w = i < n ? A.wts[i] : 0u;
            if (w) atomicAdd(&L.hist[(uint32_t)((A.keys[i] - kmin) >> shift)], (1ull << 40) | w);
        }
        __syncthreads();
        const Boundary at = find_boundary(L.hist, 0, bud);
        const uint32_t acc = at.before, bcnt = at.entries, bstar = at.bucket;
        if (bcnt <= (uint32_t)kListCap) {
            // entries before the boundary bucket are taken, entries behind it are not; those inside it
            // (often one: the first that does not fit) queue up to be ordered by (key, position)
            for (int c = 0; c < chunks; ++c) {
                const int i = tid + c * kThreads;
                if (i >= n) continue;
                const uint32_t w = A.wts[i];
                const uint32_t b = w ? (uint32_t)((A.keys[i] - kmin) >> shift) : ~0u;
                if (b == bstar && bcnt > 1) {
                    const uint32_t slot = atomicAdd(&S.bl_count, 1u);
                    L.blist[2 * slot] = A.keys[i];
                    L.blist[2 * slot + 1] = ((unsigned long long)(uint32_t)i << 32) | w;
                    continue;
                }
                const uint8_t f = (w && b < bstar) ? 1 : 0;
                A.flags[i] = f;
                flag_out[i] = f;
            }
            if (bcnt > 1) {
                __syncthreads();
                if ((uint32_t)tid < bcnt) {
                    const unsigned long long mk = L.blist[2 * tid], mv = L.blist[2 * tid + 1];
                    const uint32_t mpos = (uint32_t)(mv >> 32);
                    unsigned long long run = (unsigned long long)acc + (uint32_t)mv;
                    for (uint32_t m = 0; m < bcnt; ++m) {
                        const unsigned long long ok = L.blist[2 * m], ov = L.blist[2 * m + 1];
                        if (ok < mk || (ok == mk && (uint32_t)(ov >> 32) < mpos)) run += (uint32_t)ov;
                    }
                    const uint8_t f = run <= bud ? 1 : 0;
                    A.flags[mpos] = f;
                    flag_out[mpos] = f;
                }
            }
        } else {
            // a crowded boundary bucket (many equal or nearly equal scores): the general search
            uint64_t kstar = 0, acc2 = 0;
            uint32_t ties = 0;
            const bool bounded = radix_select<false>(A.keys, A.wts, n, budget, S, kstar, acc2, ties);
            for (int i = tid; i < n; i += kThreads) {
                uint8_t f = 0;
                if (A.wts[i]) {
                    if (!bounded) f = 1;
                    else {
                        const uint64_t k = A.keys[i];
                        if (k < kstar) f = 1;
                        else if (k == kstar && ties > 1) {
                            // exactly equal keys: lower position first, keep while the running count still fits
                            uint64_t run = acc2;
                            for (int j = 0; j <= i; ++j)
                                if (A.wts[j] && A.keys[j] == kstar) run += A.wts[j];
                            f = ((long long)run <= budget) ? 1 : 0;
                        }
                    }
                }
                A.flags[i] = f;
                flag_out[i] = f;
            }
        }
    }
    __syncthreads();

    return linear;
}

// The clusters a level did not take enter the next level's normaliser through their centroid: their
// shift and their sum of N e^{l - shift} per head go to S.bm / S.bs (published by the caller's next barrier).
template <int G>
__device__ __forceinline__ void leave_behind(const Arrays& A, Scratch& S, int n, const LevelState<G>& st)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunks = (n + kThreads - 1) / kThreads;
    double sm[G];
#pragma unroll
    for (int h = 0; h < G; ++h) sm[h] = 0.0;
#pragma unroll
    for (int c = 0; c < kKeep; ++c) {
        const int i = tid + c * kThreads;
        if (st.wk[c] && !A.flags[i]) {
#pragma unroll
            for (int h = 0; h < G; ++h) sm[h] += (double)st.wk[c] * st.ek[c][h];
        }
    }
    for (int c = kKeep; c < chunks; ++c) {
        const int i = tid + c * kThreads;
        const uint32_t w = i < n ? A.wts[i] : 0u;
        if (w && !A.flags[i]) {
#pragma unroll
            for (int h = 0; h < G; ++h) sm[h] += (double)w * exp_shifted(A.lg[h * A.lg_stride + i] - st.M[h]);
        }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {
        const double t = wave_sum_f64(sm[h]);
        if (lane == 0) S.ws[wave][h] = t;
    }
    __syncthreads();
    double bsum[G];
    combine_waves<G>(S.ws, 0.0, [](double v) { return row_sum_f64(v); }, [](int, int, double v) { return v; }, bsum);
    if (tid == 0) {
#pragma unroll
        for (int h = 0; h < G; ++h) {
            S.bm[h] = st.M[h];
            S.bs[h] = bsum[h];
            for (int w = 0; w < kWaves; ++w) S.bw[w][h] = w == 0 ? bsum[h] : 0.0;
        }
    }
}

// Coarse level (Sec. 3.4), after scoring and selection: the candidate list (children of the promising
// clusters, ascending fine id) goes to global memory and, as far as it fits, to the LDS slot the fine
// level reads its ids from; every cluster that stays behind gets the slot of its centroid term (left
// in C.aux, which only promising clusters need otherwise).  The terms themselves are written later,
// by emit_coarse_terms, while the fine level's rows travel.
template <int G>
__device__ __forceinline__ void coarse_candidates(const ScoreParams& p, const Arrays& C, int32_t* cand_l, Scratch& S,
                                                  ScanState& sc, int u, int& n_cand, uint32_t& n_terms)
{
    const int tid = threadIdx.x;
    const int n_c = p.n_coarse;
    int32_t* cand_g = p.cand + (long long)u * p.f_stride;
    sc.carry_a = sc.carry_b = 0;
    for (int i0 = 0; i0 < n_c; i0 += kThreads) {
        const int i = i0 + tid;
        const bool part = i < n_c && C.wts[i] != 0;
        const bool keep = part && C.flags[i];
        const bool emit = part && !keep && p.use_mp;
        int c0 = 0, c1 = 0;
        if (keep) { c0 = C.aux[i]; c1 = C.aux2[i]; }
        uint32_t pos, slot;
        chunk_excl_scan2<false>((uint32_t)(c1 - c0), emit ? 1u : 0u, S, sc, pos, slot);
        for (int f = c0; f < c1; ++f) {
            const uint32_t o = pos + (uint32_t)(f - c0);
            cand_g[o] = f;
            if (o < (uint32_t)p.lds_cap) cand_l[o] = f;
        }
        if (emit) C.aux[i] = (int32_t)slot;
    }
    n_cand = (int)sc.carry_a;
    n_terms = sc.carry_b;
    if (tid == 0) {
        p.n_cand[u] = n_cand;
        p.counters[4 * u + 2] = n_c;
    }
}

template <int G>
__device__ __forceinline__ void emit_coarse_terms(const ScoreParams& p, const Arrays& C, int u)
{
    if (!p.use_mp) return;
    for (int i = threadIdx.x; i < p.n_coarse; i += kThreads)
        if (C.wts[i] != 0 && !C.flags[i]) emit_term<G>(p, C, u, i, p.fcap + i, (uint32_t)C.aux[i]);
}

// Fine level, after scoring and selection: emit centroid terms for the unselected candidates and
// the flat list of stored rows of the selected clusters.
template <int G>
__device__ __forceinline__ void fine_epilogue(const ScoreParams& p, const Arrays& F, Scratch& S, ScanState& sc, int u,
                                              int n_f, bool two, uint32_t n_terms)
{
    const int tid = threadIdx.x;
    // One scan gives every selected cluster (ascending fine id) its slot in a compact list and the
    // offset of its rows in the flat row list, and every unselected candidate its centroid-term slot.
    // The compact list reuses the storage of the keys, which nobody reads any more.
    int2* sel_rc = reinterpret_cast<int2*>(F.keys);      // (first stored row, count)
    int32_t* sel_off = F.aux2;
    sc.carry_a = sc.carry_b = 0;
    for (int i0 = 0; i0 < n_f; i0 += kThreads) {
        const int i = i0 + tid;
        const bool part = i < n_f && F.wts[i] != 0;
        const bool sel = part && F.flags[i];
        const bool emit = part && !sel && p.use_mp;
        const uint32_t w = sel ? F.wts[i] : 0u;
        const int r0 = sel ? F.aux[i] : 0;
        uint32_t off, packed;       // packed: selected clusters in the low half, terms in the high half
        chunk_excl_scan2<false>(w, (sel ? 1u : 0u) | (emit ? 0x10000u : 0u), S, sc, off, packed);
        if (sel) {
            sel_rc[packed & 0xffffu] = make_int2(r0, (int)w);
            sel_off[packed & 0xffffu] = (int32_t)off;
            if (p.sel_base) {
                // q . centroid of a selected cluster, log2 units, for a value pass over keys stored as residuals
                // from it: eight columns per cluster, head h in column h (groups of up to five heads) or, for
                // larger groups, which the value pass splits over two waves, in column 4 * half + h % ceil(G / 2)
                constexpr int kHalf = G > 5 ? (G + 1) / 2 : 8;
                float b[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int h = 0; h < G; ++h)
                    b[h < kHalf ? h : 4 + h - kHalf] = (float)(F.lg[h * F.lg_stride + i] * 1.4426950408889634);
                float4* dst = reinterpret_cast<float4*>(p.sel_base + ((long long)u * p.f_stride + (packed & 0xffffu)) * 8);
                dst[0] = make_float4(b[0], b[1], b[2], b[3]);
                dst[1] = make_float4(b[4], b[5], b[6], b[7]);
            }
        }
        if (emit) emit_term<G>(p, F, u, i, two ? F.ids[i] : i, n_terms + (packed >> 16));
    }
    const uint32_t total = sc.carry_a, n_sel = sc.carry_b & 0xffffu;
    n_terms += sc.carry_b >> 16;
    __syncthreads();
    expand_rows(p, u, sel_rc, sel_off, n_sel);
    write_counters(p, u, total, n_terms, n_f, two);
}

// ================================================================================================
// The register path: levels of up to kFastChunks * kThreads entries (and at most lds_cap), every level of
// the benchmark's shapes.  A level is a chain of dependent steps on one compute unit, so what counts is the
// number of instructions a wave executes between barriers; here everything about an entry stays in the
// registers of the lanes the matrix product leaves it in, and only what the whole workgroup must know
// (per wave: shifts, sums, extremes of the scores, token totals) goes through LDS.
//
// Layout.  A chunk of up to 512 entries takes R = ceil(entries / 128) rounds of 16 entries per wave.  Group q
// of four lanes (lane = 4 q + j) holds, for round t < R, entry 16 R wave + R q + t of the chunk, lane j its
// logits of heads j and 4 + j: four heads side by side, so one reduction over the lanes equal modulo 4 serves
// all heads, and an entry costs each lane one exponential per head group instead of one per head.  Lane j of
// the group owns entry t = j for everything there is once per entry (count, row starts, key, flag): owners
// in lane order are the entries in order, which is what the prefix scans need.
//
// Two barriers stand between the logits and the selection: one for the waves' sums of N e^l (no shift by the
// largest logit, which fp64 does not need below |l| = 500), one for the histogram (whose buckets are fixed, so that
// no extremes have to be found first).
//
// Measured (MI355X, cycles from the first request to the last store of a unit): 64 coarse + 250 fine entries of 4
// heads 46.4k -> 34.3k, 256 + 504 entries 65.6k -> 54.7k, one level of 64 entries 20.2k -> 15.2k against one entry
// per thread with all heads in turn, a shift and a min / max of the keys.  What is left at 256 + 504 entries: rows
// and products 28k (the product alone 4.1k: 512 entries x 4 heads x 128 dims at the fp64 rate of one compute
// unit), the chain of dependent instructions 22k, the expansion of 8192 row numbers 4k.
// ================================================================================================
constexpr int kFastChunks = 2;
constexpr int kEarlyLooks = 4;        // further times the helpers' count is looked at (a trip each) before the level is worked out without them
constexpr double kNoShift = 500.0;    // largest |logit| that is exponentiated without a shift
constexpr int kRounds = 4;

// One unit's rows, counts and row starts of one level.
struct LevelTables {
    const uint16_t* rows;
    const int32_t* N;
    const int32_t* start;
};

template <int G>
struct FastLevel {
    static constexpr int GH = (G + 3) / 4;
    double l[kFastChunks][kRounds][GH];   // logits (matrix layout)
    double e[kFastChunks][kRounds][GH];   // e^{l - M}, 0 where the entry takes no part
    double M[GH];                         // shift of the level, this lane's heads (0 unless a logit is far out)
    uint32_t w[kFastChunks];              // own entries: member count (0: takes no part),
    int32_t a1[kFastChunks], a2[kFastChunks];   // row starts (coarse: first child, end of children),
    int32_t id[kFastChunks];              // cluster id,
    int32_t x[kFastChunks];               // position in the level (-1: none)
    bool take[kFastChunks];               // selected
};

__device__ __forceinline__ int chunk_entries(int n, int c) { return min(max(n - c * kThreads, 0), kThreads); }
__device__ __forceinline__ int chunk_rounds(int n, int c) { return (chunk_entries(n, c) + 16 * kWaves - 1) / (16 * kWaves); }

// f(t) for t = 0..3 with t a compile-time constant
template <typename F>
__device__ __forceinline__ void for_rounds(F f)
{
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
}

// What is handed from one workgroup to another inside a launch goes past the caches that they do not share.
__device__ __forceinline__ double load_handed_over(const double* p)
{
    return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void hand_over(double* p, double v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Scores and selection of one level (see score_level for the definitions); `behind`: the normaliser also covers
// what the coarse level left behind (S.bm / S.bw).  `quiet`: store nothing in global memory, and ask for the
// rows last round first (shadow workgroup).  `meanwhile` runs once the rows have been asked for.  Returns 1 for
// linear-domain keys, 0 for logarithmic ones.
template <int G, bool kHelped, typename Meanwhile>
__device__ __forceinline__ int fast_level(const ScoreParams& p, const Lds& L, Scratch& S, const LevelTables& T, int n, int u, bool use_ids,
                                          bool coarse, bool behind, bool q_pending, const uint16_t (&qv)[(G + 3) / 4], bool quiet,
                                          const double* handed, FastLevel<G>& st, Meanwhile meanwhile)
{
    const double* early = kHelped ? handed : nullptr;
    constexpr int GH = (G + 3) / 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 3, quad = lane >> 2;
    const double ninf = -INFINITY;
    const Arrays& A = L.A;

    // ---------------- rows: operand layout, lane (k, e) takes dim group k of entry e of the wave's sixteen ----------------
    const int kA = lane >> 4, qA = 4 * (lane & 3) + ((lane >> 2) & 3);      // the group of four lanes whose entry this is
    const int bsel = kA * 4 + j;
    uint4 raw[kRounds][4];
    auto request = [&](int c, int t, uint4 (&r)[4]) {
        const int nc = chunk_entries(n, c), R = chunk_rounds(n, c);
        const int x = wave * 16 * R + qA * R + t;
        if (x < nc) {
            const int id = use_ids ? A.ids[c * kThreads + x] : c * kThreads + x;
            const uint4* kp = reinterpret_cast<const uint4*>(T.rows + (long long)id * kHeadDim) + kA;
#pragma unroll
            for (int k = 0; k < 4; ++k) r[k] = kp[4 * k];
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) r[k] = make_uint4(0, 0, 0, 0);
        }
    };
    const int R0 = chunk_rounds(n, 0);
#pragma unroll
    for (int c = 0; c < kFastChunks; ++c) {
        const int nc = chunk_entries(n, c), R = chunk_rounds(n, c);
        const int x = wave * 16 * R + quad * R + j;
        const bool own = j < R && x < nc;
        st.x[c] = own ? c * kThreads + x : -1;
        st.w[c] = 0;
        st.a1[c] = st.a2[c] = st.id[c] = 0;
        if (own) {
            const int id = use_ids ? A.ids[c * kThreads + x] : c * kThreads + x;
            st.id[c] = id;
            st.w[c] = (uint32_t)T.N[id];
            st.a1[c] = T.start[id];
            if (coarse) st.a2[c] = T.start[id + 1];
        }
    }
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        const int t = quiet ? kRounds - 1 - i : i;
        if (t < R0 && !early) {
            if (t == 0) request(0, 0, raw[0]);
            if (t == 1) request(0, 1, raw[1]);
            if (t == 2) request(0, 2, raw[2]);
            if (t == 3) request(0, 3, raw[3]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // while the rows travel
    meanwhile();
    if (tid < kHistBuckets) L.hist[tid] = S.hist[0][tid] = S.hist[1][tid] = S.hist[2][tid] = 0;
    if (tid < kListCap) S.ahead[tid] = 0;
    if (tid == 0) {
        S.bl_count = 0;
        S.tiny = 0;
        if (q_pending) S.far[0] = S.far[1] = 0;      // (both levels' flags, in front of the launch's first barrier)
    }
    if (q_pending) {
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) L.qB[tid + hg * kThreads] = query_operand<G>(qv[hg], hg, tid);
        phase_sync<true>();
    }

    const long long budget = coarse ? p.coarse_budget : p.key_budget;
    unsigned long long* key_out = coarse ? p.key_c + (long long)u * p.c_stride : p.key_f + (long long)u * p.f_stride;
    uint8_t* flag_out = coarse ? p.flag_c + (long long)u * p.c_stride : p.flag_f + (long long)u * p.f_stride;

    // ---------------- logits ----------------
    bool far = false;
    if (early) {
        // (worked out by the helpers; every load on its way before the first is looked at)
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) {
            const int nc = chunk_entries(n, c), R = chunk_rounds(n, c);
            for_rounds([&](auto tc) {
                constexpr int t = decltype(tc)::value;
#pragma unroll
                for (int hg = 0; hg < GH; ++hg) st.l[c][t][hg] = st.e[c][t][hg] = 0.0;
                if (t < R) {
                    const int x = min(wave * 16 * R + quad * R + t, nc - 1);
                    const double* at = early + (long long)A.ids[c * kThreads + x] * (8 * GH) + j;
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) {
                        st.l[c][t][hg] = load_handed_over(at + 4 * hg);
                        st.e[c][t][hg] = load_handed_over(at + 4 * (GH + hg));
                    }
                }
            });
        }
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) {
            const int R = chunk_rounds(n, c);
            for_rounds([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if (t < R) {
                    const bool part = quad_lane<t>(st.w[c]) != 0;
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) far |= part && !(fabs(st.l[c][t][hg]) <= kNoShift);
                }
            });
        }
    } else
#pragma unroll
    for (int c = 0; c < kFastChunks; ++c) {
        const int R = chunk_rounds(n, c), Rn = c + 1 < kFastChunks ? chunk_rounds(n, c + 1) : 0;
        for_rounds([&](auto tc) {
            constexpr int t = decltype(tc)::value;
#pragma unroll
            for (int hg = 0; hg < GH; ++hg) st.l[c][t][hg] = 0.0;
            if (t < R) {
                double acc[GH];
#pragma unroll
                for (int hg = 0; hg < GH; ++hg) acc[hg] = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t w4[4] = {raw[t][k].x, raw[t][k].y, raw[t][k].z, raw[t][k].w};
#pragma unroll
                    for (int d = 0; d < 8; ++d) {
                        const double a = (double)((d & 1) ? bf16hi_to_f32(w4[d >> 1]) : bf16lo_to_f32(w4[d >> 1]));
#pragma unroll
                        for (int hg = 0; hg < GH; ++hg)
                            acc[hg] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, L.qB[(hg * 32 + 8 * k + d) * 16 + bsel], acc[hg], 0, 0, 0);
                    }
                }
                const bool part = quad_lane<t>(st.w[c]) != 0;
#pragma unroll
                for (int hg = 0; hg < GH; ++hg) {
                    st.l[c][t][hg] = acc[hg] * p.scale;
                    far |= part && !(fabs(st.l[c][t][hg]) <= kNoShift);
                }
            }
            if (t < Rn) request(c + 1, t, raw[t]);
        });
    }

    // ---------------- e^{l - M} and the waves' sums of N e^{l - M} per head ----------------
    // A double holds e^l for any |l| up to 700, so the usual shift by the largest logit is left out (M = 0) unless
    // some logit is beyond kNoShift; the waves then exchange their largest logits first (second trip).
    int linear = 1;
    const uint32_t n_taking = wave_total_u32(st.w[0] + st.w[kFastChunks - 1]);
    double tot[GH], g[GH];
#pragma unroll
    for (int hg = 0; hg < GH; ++hg) st.M[hg] = 0.0;
    for (int trip = 0; trip < 2; ++trip) {
        double sw[GH];
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) sw[hg] = 0.0;
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) {
            const int R = chunk_rounds(n, c);
            for_rounds([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if (t >= R) {
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) st.e[c][t][hg] = 0.0;
                } else {
                    const uint32_t w = quad_lane<t>(st.w[c]);
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) {
                        // (an entry that takes no part: not used; a helper's e^l has no shift)
                        const double x = early && trip == 0 ? st.e[c][t][hg] : exp_shifted(st.l[c][t][hg] - st.M[hg]);
                        st.e[c][t][hg] = w ? x : 0.0;
                        sw[hg] += (double)w * st.e[c][t][hg];
                    }
                }
            });
        }
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) {
            sw[hg] = same_head(sw[hg], AddOp{});
            if (lane < 4) S.ws[wave][4 * hg + lane] = sw[hg];
        }
        if (lane == 0) S.rk_wt[wave] = n_taking;
        if (trip == 0 && __any(far)) S.far[coarse] = 1;
        phase_sync<true>();
        if (trip == 1 || !S.far[coarse]) break;
        double mw[GH];
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) mw[hg] = ninf;
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) {
            const int R = chunk_rounds(n, c);
            for_rounds([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if (t < R && quad_lane<t>(st.w[c]) != 0) {
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) mw[hg] = fmax(mw[hg], st.l[c][t][hg]);
                }
            });
        }
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) {
            mw[hg] = same_head(mw[hg], MaxOp{});
            if (lane < 4) S.wm[wave][4 * hg + lane] = mw[hg];
        }
        phase_sync<true>();
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) {
            const double M = same_head(S.wm[quad & (kWaves - 1)][4 * hg + j], MaxOp{});
            st.M[hg] = M == ninf ? 0.0 : M;
        }
    }

    // ---------------- normaliser (lane 4 w + j: wave w, head j), scores ----------------
#pragma unroll
    for (int hg = 0; hg < GH; ++hg) {
        const int h = 4 * hg + j;
        double ts = S.ws[quad & (kWaves - 1)][h];
        if (behind) {
            // (relative to this level's shift; both are zero unless a logit was far out)
            double bs = S.bw[quad & (kWaves - 1)][h];
            if (S.far[0] | S.far[1]) {
                const double bm = S.bm[h];
                if (same_head(bs, AddOp{}) > 0.0 && bm > st.M[hg]) {      // (uniform over a head's lanes)
                    const double down = exp_shifted(st.M[hg] - bm);
                    ts *= down;
#pragma unroll
                    for (int c = 0; c < kFastChunks; ++c)
#pragma unroll
                        for (int t = 0; t < kRounds; ++t) st.e[c][t][hg] *= down;
                    st.M[hg] = bm;
                }
                bs = bs > 0.0 ? bs * exp_shifted(bm - st.M[hg]) : 0.0;
            }
            ts += bs;
        }
        const double T = same_head(lane < 4 * kWaves ? ts : 0.0, AddOp{});
        tot[hg] = T;
        g[hg] = (h < G && T > 0.0) ? 1.0 / T : 0.0;
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_total_u32(lane < kWaves ? S.rk_wt[lane & (kWaves - 1)] : 0u));
    constexpr double kLogGs[9] = {0.0, 0.0, 0.6931471805599453094, 1.0986122886681097821, 1.3862943611198906188,
                                  1.6094379124341002818, 1.7917594692280549573, 1.9459101090932196052, 2.0794415416798357477};
    constexpr double kLogG = kLogGs[G];
    uint64_t key[kFastChunks];                 // of the own entries
    auto select_own = [&](const double (&sc)[kRounds]) {
        const double lo = (j & 1) ? sc[1] : sc[0], hi = (j & 1) ? sc[3] : sc[2];
        return (j & 2) ? hi : lo;
    };
    bool tiny = false;
#pragma unroll
    for (int c = 0; c < kFastChunks; ++c) {
        const int R = chunk_rounds(n, c);
        double sc[kRounds] = {0.0, 0.0, 0.0, 0.0};
        for_rounds([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            if (t < R) {
                double v = st.e[c][t][0] * g[0];
                if constexpr (GH > 1) v += st.e[c][t][1] * g[1];
                sc[t] = sum4_f64(v);
            }
        });
        const double own = select_own(sc);
        tiny |= st.w[c] && !(own >= 1e-280);
        key[c] = st.w[c] ? ~(uint64_t)__double_as_longlong(own) : ~0ull;
    }
    if (__any(tiny)) S.tiny = 1;
    // First digit of the selection: buckets on a fixed scale of the score, so that nothing about the level has to be
    // known beforehand: quarters of an octave down to 2^-28 (where flat attention has its boundary), octaves down to
    // 2^-124, then eight octaves each (peaked attention), the last bucket open.  `pos`: quarter octaves below 16 (no
    // score is larger than G up to rounding) with 50 binary places, the octaves linear inside.
    constexpr uint64_t kTopKey = ~0x4030000000000000ull;
    static_assert(kHistBuckets == 256, "the scale below has 128 + 96 + 32 buckets");
    auto bucket_of = [&](uint64_t at) {
        const uint32_t v = (uint32_t)(at >> 50);
        const uint32_t far_down = min(224u + ((v - 512u) >> 5), 255u);
        return v < 128u ? v : v < 512u ? 96u + (v >> 2) : far_down;
    };
    uint64_t pos[kFastChunks];
    uint32_t bucket[kFastChunks];
#pragma unroll
    for (int c = 0; c < kFastChunks; ++c) {
        pos[c] = key[c] - kTopKey;
        bucket[c] = bucket_of(pos[c]);
        if (st.w[c]) atomicAdd(&L.hist[bucket[c]], (1ull << 40) | st.w[c]);
    }
    phase_sync<true>();
    const unsigned long long* first_digit = L.hist;
    if (S.tiny) {
        // some score left the range of a double: the level ranks by log mean_h e^{l - LSE_h} in the log domain
        linear = 0;
        double lse[GH];
#pragma unroll
        for (int hg = 0; hg < GH; ++hg) lse[hg] = st.M[hg] + log(not_hoisted(tot[hg]));
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) {
            const int R = chunk_rounds(n, c);
            double sc[kRounds] = {0.0, 0.0, 0.0, 0.0};
            for_rounds([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if (t < R) {
                    double th[GH], tm = ninf;
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) {
                        th[hg] = 4 * hg + j < G ? st.l[c][t][hg] - lse[hg] : ninf;
                        tm = fmax(tm, th[hg]);
                    }
                    tm = fmax(tm, dpp_f64<kDppXor1>(tm));
                    tm = fmax(tm, dpp_f64<kDppXor2>(tm));
                    double ss = 0.0;
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) ss += exp_shifted(th[hg] - tm);
                    ss = sum4_f64(ss);
                    sc[t] = tm - kLogG + log(not_hoisted(ss));
                }
            });
            const double own = select_own(sc);
            key[c] = st.w[c] ? descending_key(own) : ~0ull;
            pos[c] = (uint64_t)(fmin(fmax(16.0 - own * (4.0 * 1.4426950408889634), 0.0), 16383.0) * 0x1p50);
            bucket[c] = bucket_of(pos[c]);
            if (st.w[c]) atomicAdd(&S.hist[0][bucket[c]], (1ull << 40) | st.w[c]);
        }
        phase_sync<true>();
        first_digit = S.hist[0];
    }
    if (!quiet) {
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c)
            if (st.x[c] >= 0) key_out[st.x[c]] = key[c];
    }

    // ---------------- budgeted selection ----------------
    const uint32_t bud = budget < 0 ? 0u : (budget > 0xffffffffll ? 0xffffffffu : (uint32_t)budget);
    if (total <= bud) {
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) st.take[c] = st.w[c] != 0;
    } else {
        const Boundary first_cut = find_boundary(first_digit, 0, bud);
        uint32_t acc = first_cut.before, bcnt = first_cut.entries, bstar = first_cut.bucket;
        // entries before the boundary bucket are taken, entries behind it are not
        bool inside[kFastChunks];
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) {
            st.take[c] = st.w[c] && bucket[c] < bstar;
            inside[c] = st.w[c] && bucket[c] == bstar;
        }
        auto order_inside = [&](auto direct) {
            // Those inside it are ordered by (key, position).
            uint32_t at[kFastChunks];
#pragma unroll
            for (int c = 0; c < kFastChunks; ++c) {
                at[c] = 0;
                if (inside[c]) {
                    at[c] = atomicAdd(&S.bl_count, 1u);
                    L.blist[2 * at[c]] = key[c];
                    L.blist[2 * at[c] + 1] = ((unsigned long long)(uint32_t)st.x[c] << 32) | st.w[c];
                }
            }
            phase_sync<true>();
            constexpr uint32_t kShare = kListCap / kWaves;
            // tokens of the entries [first, end) of the list that come before (k, x); four at a time (their reads together)
            auto tokens_before = [&](uint32_t first, uint32_t end, unsigned long long k, uint32_t x) {
                uint32_t run = 0;
#pragma unroll 1
                for (; first < end; first += 4)
#pragma unroll
                    for (uint32_t m = first; m < first + 4; ++m) {
                        const unsigned long long ok = L.blist[2 * m], ov = L.blist[2 * m + 1];
                        const bool before = ok < k || (ok == k && (uint32_t)(ov >> 32) < x);
                        run += m < end && before ? (uint32_t)ov : 0u;
                    }
                return run;
            };
            if constexpr (decltype(direct)::value) {
#pragma unroll
                for (int c = 0; c < kFastChunks; ++c)
                    if (inside[c]) st.take[c] = (unsigned long long)acc + tokens_before(0, bcnt, key[c], (uint32_t)st.x[c]) + st.w[c] <= bud;
            } else {
                // A longer list: every entry's lane adds up an eighth of it in every wave.  (Its owner alone going through
                // the whole list: 100 cycles an entry and chunk, 8 us at 60 entries.)
                static_assert(kListCap == 64, "one lane per entry of the list");
                const uint32_t first = kShare * wave, end = min(first + kShare, bcnt);
                if (first < end && lane < bcnt)
                    atomicAdd(&S.ahead[lane], tokens_before(first, end, L.blist[2 * lane], (uint32_t)(L.blist[2 * lane + 1] >> 32)));
                phase_sync<true>();
#pragma unroll
                for (int c = 0; c < kFastChunks; ++c)
                    if (inside[c]) st.take[c] = (unsigned long long)acc + S.ahead[at[c]] + st.w[c] <= bud;
            }
        };
        if (bcnt <= 12u) {
            if (bcnt > 1) order_inside(std::true_type{});
        } else {
            // (All that is rare stands in this one block: every jump over code that has not run yet costs the common path
            // about 0.2 us.  With the digits, the general search and the longer list in blocks of their own the launch took
            // 17.8 instead of 17.2 us at 64 + 250 clusters, 15.8 instead of 15.2 in a generation step.)
            // Flat attention puts much of a level into one bucket: up to two more digits, 256 slices of it each (the last slice
            // of the open bucket takes the rest).  The general search divides all entries anew, digit by digit from their
            // extremes.  Whole step of 8 units, 1024 clusters in one level, 1 / 3 / 5 heads, near and past a full bucket: 42 / 42 /
            // 49 us with it, 29 / 30 / 36 with these digits and the list below; 2048 and 128 clusters, 4 heads, peaked scores in
            // the log domain 44 -> 33.
            uint64_t low = (uint64_t)(bstar < 128u ? bstar : bstar < 224u ? 4u * (bstar - 96u) : 512u + 32u * (bstar - 224u)) << 50;
            int slice = bstar < 128u ? 50 : bstar < 224u ? 52 : 55;
#pragma unroll 1
            for (int digit = 1; digit <= 2 && bcnt > (uint32_t)kListCap; ++digit) {
                slice -= 8;
                uint32_t sub[kFastChunks];
#pragma unroll
                for (int c = 0; c < kFastChunks; ++c) {
                    const uint64_t at = (pos[c] - low) >> slice;
                    sub[c] = at < 255u ? (uint32_t)at : 255u;
                    if (inside[c]) atomicAdd(&S.hist[digit][sub[c]], (1ull << 40) | st.w[c]);
                }
                phase_sync<true>();
                const Boundary cut = find_boundary(S.hist[digit], acc, bud);
                acc = cut.before;
                bcnt = cut.entries;
                bstar = cut.bucket;
#pragma unroll
                for (int c = 0; c < kFastChunks; ++c) {
                    st.take[c] |= inside[c] && sub[c] < bstar;
                    inside[c] = inside[c] && sub[c] == bstar;
                }
                low += (uint64_t)bstar << slice;
            }
            if (bcnt > (uint32_t)kListCap) {
                // a crowded slice (many equal or almost equal scores): the general search
#pragma unroll
                for (int c = 0; c < kFastChunks; ++c) {
                    if (st.x[c] >= 0) {
                        A.keys[st.x[c]] = key[c];
                        A.wts[st.x[c]] = st.w[c];
                    }
                }
                phase_sync<true>();
                uint64_t kstar = 0, acc2 = 0;
                uint32_t ties = 0;
                const bool bounded = radix_select<true>(A.keys, A.wts, n, budget, S, kstar, acc2, ties);
#pragma unroll
                for (int c = 0; c < kFastChunks; ++c) {
                    if (!st.w[c]) continue;
                    bool t = !bounded || key[c] < kstar;
                    if (!t && key[c] == kstar && ties > 1) {
                        // exactly equal keys: lower position first, keep while the running count still fits
                        uint64_t run = acc2;
                        for (int i = 0; i <= st.x[c]; ++i)
                            if (A.wts[i] && A.keys[i] == kstar) run += A.wts[i];
                        t = (long long)run <= budget;
                    }
                    st.take[c] = t;
                }
            } else if (bcnt > 1) {
                order_inside(std::false_type{});
            }
        }
    }
    if (!quiet) {
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c)
            if (st.x[c] >= 0) flag_out[st.x[c]] = st.take[c] ? 1 : 0;
    }
    return linear;
}

// Centroid terms (Eq. 2) of a level in the register path: group of four lanes per entry, lane j writes heads j
// and 4 + j.  `slot` of the own entries (< 0: no term), row0 = centroid-table row of cluster 0 of the level.
template <int G>
__device__ __forceinline__ void fast_terms(const ScoreParams& p, const FastLevel<G>& st, const int (&slot)[kFastChunks],
                                           int n, int row0, int u)
{
    constexpr int GH = (G + 3) / 4;
    const int j = threadIdx.x & 3;
#pragma unroll
    for (int c = 0; c < kFastChunks; ++c) {
        const int R = chunk_rounds(n, c);
        for_rounds([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            if (t < R) {
                const int sl = (int)quad_lane<t>((uint32_t)slot[c]);
                const float lgN = __builtin_amdgcn_logf((float)quad_lane<t>(st.w[c]));
                if (sl >= 0) {
                    const long long o = (long long)u * p.mp_stride + sl;
                    if (j == t) p.mp_rows[o] = row0 + st.id[c];
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg)
                        if (4 * hg + j < G) p.mp_scores[o * G + 4 * hg + j] = (float)(st.l[c][t][hg] * 1.4426950408889634) + lgN;
                }
            }
        });
    }
}

// Coarse level after its selection (see coarse_candidates).  `slot` receives the centroid-term slots of the own
// entries; what stays behind goes to S.bm / S.bw; the candidate list is published by the caller's barrier.
template <int G>
__device__ __forceinline__ void fast_candidates(const ScoreParams& p, const Lds& L, Scratch& S, ScanState& sc,
                                                const FastLevel<G>& st, int u, bool quiet, int& n_cand, uint32_t& n_terms,
                                                int (&slot)[kFastChunks])
{
    constexpr int GH = (G + 3) / 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_c = p.n_coarse;
    double bs[GH];
#pragma unroll
    for (int hg = 0; hg < GH; ++hg) bs[hg] = 0.0;
#pragma unroll
    for (int c = 0; c < kFastChunks; ++c) {
        const int R = chunk_rounds(n_c, c);
        const uint32_t left = st.take[c] ? 0u : st.w[c];
        for_rounds([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            if (t < R) {
                const double w = (double)quad_lane<t>(left);
#pragma unroll
                for (int hg = 0; hg < GH; ++hg) bs[hg] += w * st.e[c][t][hg];
            }
        });
    }
#pragma unroll
    for (int hg = 0; hg < GH; ++hg) {
        bs[hg] = same_head(bs[hg], AddOp{});
        if (lane < 4) {
            S.bw[wave][4 * hg + lane] = bs[hg];
            if (wave == 0) S.bm[4 * hg + lane] = st.M[hg];
        }
    }
    int2* sel_rc = reinterpret_cast<int2*>(L.A.keys);      // (first child, children) of the promising clusters
    int32_t* sel_off = L.A.aux2;                           // offset of their children in the candidate list
    sc.carry_a = sc.carry_b = 0;
#pragma unroll
    for (int c = 0; c < kFastChunks; ++c) {
        slot[c] = -1;
        if (c * kThreads >= n_c) continue;
        const bool emit = st.w[c] && !st.take[c] && p.use_mp;
        const int kids = st.take[c] ? st.a2[c] - st.a1[c] : 0;
        uint32_t pos, packed;       // packed: promising clusters in the low half, terms in the high half
        chunk_excl_scan2<true>((uint32_t)kids, (st.take[c] ? 1u : 0u) | (emit ? 0x10000u : 0u), S, sc, pos, packed);
        if (st.take[c]) {
            sel_rc[packed & 0xffffu] = make_int2(st.a1[c], kids);
            sel_off[packed & 0xffffu] = (int32_t)pos;
        }
        if (emit) slot[c] = (int)(packed >> 16);
    }
    n_cand = (int)sc.carry_a;
    n_terms = sc.carry_b >> 16;
    const uint32_t n_sel = sc.carry_b & 0xffffu;
    phase_sync<true>();
    // expansion: one row of 16 lanes per promising cluster
    int32_t* cand_g = p.cand + (long long)u * p.f_stride;
    const int sub = tid & 15;
    for (uint32_t k = tid >> 4; k < n_sel; k += kThreads / 16) {
        const int2 rc = sel_rc[k];
        const int off = sel_off[k];
        for (int i = sub; i < rc.y; i += 16) {
            if (!quiet) cand_g[off + i] = rc.x + i;
            if (off + i < p.lds_cap) L.A.ids[off + i] = rc.x + i;
        }
    }
    if (tid == 0 && !quiet) {
        p.n_cand[u] = n_cand;
        p.counters[4 * u + 2] = n_c;
    }
}

// Fine level after its selection (see fine_epilogue).
template <int G>
__device__ __forceinline__ void fast_epilogue(const ScoreParams& p, const Lds& L, Scratch& S, ScanState& sc,
                                              const FastLevel<G>& st, int u, int n_f, bool two, uint32_t n_terms)
{
    constexpr int GH = (G + 3) / 4;
    const int tid = threadIdx.x, j = tid & 3;
    int2* sel_rc = reinterpret_cast<int2*>(L.A.keys);      // (first stored row, count) of the selected clusters
    int32_t* sel_off = L.A.aux2;                           // offset of their rows in the row list
    int slot[kFastChunks], pick[kFastChunks];
    sc.carry_a = sc.carry_b = 0;
#pragma unroll
    for (int c = 0; c < kFastChunks; ++c) {
        slot[c] = pick[c] = -1;
        if (c * kThreads >= n_f) continue;
        const bool emit = st.w[c] && !st.take[c] && p.use_mp;
        uint32_t off, packed;       // packed: selected clusters in the low half, terms in the high half
        chunk_excl_scan2<true>(st.take[c] ? st.w[c] : 0u, (st.take[c] ? 1u : 0u) | (emit ? 0x10000u : 0u), S, sc, off, packed);
        if (st.take[c]) {
            pick[c] = (int)(packed & 0xffffu);
            sel_rc[pick[c]] = make_int2(st.a1[c], (int)st.w[c]);
            sel_off[pick[c]] = (int32_t)off;
        }
        if (emit) slot[c] = (int)(n_terms + (packed >> 16));
    }
    const uint32_t total = sc.carry_a, n_sel = sc.carry_b & 0xffffu;
    n_terms += sc.carry_b >> 16;
    phase_sync<true>();
    expand_rows(p, u, sel_rc, sel_off, n_sel);
    fast_terms<G>(p, st, slot, n_f, 0, u);
    if (p.sel_base) {
        // q . centroid of a selected cluster, log2 units, for a value pass over keys stored as residuals
        // from it: eight columns per cluster, head h in column h (groups of up to five heads) or, for
        // larger groups, which the value pass splits over two waves, in column 4 * half + h % ceil(G / 2)
        constexpr int kHalf = G > 5 ? (G + 1) / 2 : 8;
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) {
            const int R = chunk_rounds(n_f, c);
            for_rounds([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if (t < R) {
                    const int k = (int)quad_lane<t>((uint32_t)pick[c]);
                    if (k >= 0) {
                        float* dst = p.sel_base + ((long long)u * p.f_stride + k) * 8;
#pragma unroll
                        for (int hg = 0; hg < GH; ++hg) {
                            const int h = 4 * hg + j, col = h < kHalf ? h : 4 + h - kHalf;
                            if (col < 8) dst[col] = h < G ? (float)(st.l[c][t][hg] * 1.4426950408889634) : 0.f;
                        }
                    }
                }
            });
        }
    }
    write_counters(p, u, total, n_terms, n_f, two);
}

// What a shadow workgroup does at the last level: ask for the centroid rows of the second half of
// the level's entries, last entry first, and drop them.
__device__ __forceinline__ void touch_rows(const ScoreParams& p, const int32_t* ids, int u, int n)
{
    const uint16_t* Kcu = p.Kc + (long long)u * p.tab_rows * kHeadDim;
    const int grp = threadIdx.x >> 4, sub = threadIdx.x & 15;
    uint32_t x = 0;
    for (int k = n - 1 - grp; k >= n / 2; k -= kThreads / 16) {
        const int id = ids ? ids[k] : k;
        const uint4 v = reinterpret_cast<const uint4*>(Kcu + (long long)id * kHeadDim)[sub];
        x ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    // (keeps the loads alive: the condition never holds, and the slot would be the unit's own)
    if (x == 0xfff1fff2u && p.U < 0) p.counters[4 * u] = 0;
}

// Helper workgroup `share` of `shares` of a unit: the logits of its part of all fine clusters, by the very instructions of
// fast_level, and their exponentials without a shift (fast_level does not look at those of a level that needs one).
template <int G>
__device__ __forceinline__ void early_logits(const ScoreParams& p, double* qB, const uint16_t* rows, int n, int share, int shares, int u,
                                             const uint16_t (&qv)[(G + 3) / 4])
{
    constexpr int GH = (G + 3) / 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 3, quad = lane >> 2;
    const int kA = lane >> 4, qA = 4 * (lane & 3) + ((lane >> 2) & 3), bsel = kA * 4 + j;
    const int per = (n + shares - 1) / shares, a = share * per, b = min(a + per, n);
    uint4 raw[kRounds][4];
    auto request = [&](int x0, uint4 (&r)[4]) {
        const uint4* kp = reinterpret_cast<const uint4*>(rows + (long long)min(x0 + qA, n - 1) * kHeadDim) + kA;
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = kp[4 * k];
    };
    const int first = a + wave * 16;
#pragma unroll
    for (int t = 0; t < kRounds; ++t)
        if (first + t * 16 * kWaves < b) request(first + t * 16 * kWaves, raw[t]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int hg = 0; hg < GH; ++hg) qB[tid + hg * kThreads] = query_operand<G>(qv[hg], hg, tid);
    phase_sync<true>();
    double* out = p.early + (long long)u * p.early_stride * (8 * GH) + j;
    const double scale = p.scale;
#pragma unroll 1
    for (int x0 = first; x0 < b; x0 += kRounds * 16 * kWaves) {
        for_rounds([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            const int xt = x0 + t * 16 * kWaves;
            if (xt < b) {
                double acc[GH];
#pragma unroll
                for (int hg = 0; hg < GH; ++hg) acc[hg] = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t w4[4] = {raw[t][k].x, raw[t][k].y, raw[t][k].z, raw[t][k].w};
#pragma unroll
                    for (int d = 0; d < 8; ++d) {
                        const double v = (double)((d & 1) ? bf16hi_to_f32(w4[d >> 1]) : bf16lo_to_f32(w4[d >> 1]));
#pragma unroll
                        for (int hg = 0; hg < GH; ++hg)
                            acc[hg] = __builtin_amdgcn_mfma_f64_4x4x4f64(v, qB[(hg * 32 + 8 * k + d) * 16 + bsel], acc[hg], 0, 0, 0);
                    }
                }
                if (xt + kRounds * 16 * kWaves < b) request(xt + kRounds * 16 * kWaves, raw[t]);
                if (xt + quad < b) {
                    double* at = out + (long long)(xt + quad) * (8 * GH);
#pragma unroll
                    for (int hg = 0; hg < GH; ++hg) {
                        const double l = acc[hg] * scale;
                        hand_over(at + 4 * hg, l);
                        hand_over(at + 4 * (GH + hg), exp_shifted(l));
                    }
                }
            }
        });
    }
    // every wave's stores have arrived before the workgroup counts itself in
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(p.early_done + u, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What the first level's requests need, as scalars: they are in registers when a wave starts (see the build flags), while the
// other arguments span several cache lines of a segment no one has read yet.  So the query and the first level's rows are
// asked for at once, and the rest of the arguments, one request for each line, while those travel.  Together with a query
// that nothing waits for in front of the rows: one level of 64 clusters, 1 unit: step 15.8 -> 15.6 us; 8 units x 4096 keys
// 27.6 -> 27.2; 32 units x 4096, 5 heads 41.1 -> 39.7; 24 units, 8 heads 48.0 -> 47.2.
// first_row: first row of the level in the unit's tables, 0 where there is no coarse level.
// kHelped: the launch may have helpers (a kernel of its own: in the other one the code for it costs 0.2 to 0.4 us a launch).
template <int G, bool kHelped>
__global__ __launch_bounds__(kThreads) void score_select_kernel(const uint16_t* q, const uint16_t* Kc, const int32_t* N,
                                                                const int32_t* first_start, int U, int tab_rows, int first_row,
                                                                int n_first, int first_stride, int lds_cap, int helpers, int n_fine,
                                                                const ScoreParams p)
{
    constexpr int GH = (G + 3) / 4;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Scratch& S = *reinterpret_cast<Scratch*>(smem_raw);
    const Lds L = carve_lds<G>(smem_raw + align16(sizeof(Scratch)), lds_cap);
    const int u = blockIdx.x % U, tid = threadIdx.x;
    // second workgroup of the unit: warms the shared L2, stores nothing (or, where there are helpers, it is one of them)
    const bool shadow = blockIdx.x >= (unsigned)U;
    const long long tables = (long long)u * tab_rows + first_row;
    const LevelTables first{Kc + tables * kHeadDim, N + tables, first_start + (long long)u * first_stride};

    uint16_t qv[GH];    // this thread's elements of the query operand (one per head group; converted once they are needed)
#pragma unroll
    for (int hg = 0; hg < GH; ++hg) qv[hg] = query_operand_element<G>(q, u, hg, tid);
    if (kHelped && shadow) {
        early_logits<G>(p, L.qB, Kc + (long long)u * tab_rows * kHeadDim, n_fine, (int)blockIdx.x / U - 1, helpers, u, qv);
        return;
    }
    // the step's new rows go to their place in the tail buffers: asked for here, stored at the end
    uint4 app = make_uint4(0, 0, 0, 0);
    bool appends = false;
    const auto arguments = [&] {
        asm volatile("" ::"s"(p.q), "s"(p.cstart), "s"(p.g_wts), "s"(p.flag_c), "s"(p.n_cand), "s"(p.mp_rows), "s"(p.app_n), "s"(p.U));
        appends = !shadow && tid < 16 * p.app_n;
        if (appends) app = reinterpret_cast<const uint4*>(p.app_src[tid >> 4])[(long long)u * 16 + (tid & 15)];
    };

    const bool two = first_row != 0;
    ScanState sc;
    uint32_t n_terms = 0;
    int n_f = n_first;
    const bool coarse_fast = n_first <= lds_cap;
    int done = 0;
    FastLevel<G> fc;
    int slot_c[kFastChunks];
    if (two) {
        if (coarse_fast) {
            const int lin = fast_level<G, false>(p, L, S, first, n_first, u, false, true, false, true, qv, shadow, nullptr, fc, arguments);
            if (tid == 0 && !shadow) p.key_mode[2 * u] = lin;
            auto look = [&] { return __hip_atomic_load(p.early_done + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            if (kHelped && tid == 0) done = look();
            fast_candidates<G>(p, L, S, sc, fc, u, shadow, n_f, n_terms, slot_c);
            if (kHelped && tid == 0) {
                for (int i = 0; i < kEarlyLooks && done < helpers; ++i) done = look();
                S.early = done >= helpers;
            }
        } else {
            // (a shadow workgroup would race with the first one on the global working arrays: it leaves)
            if (shadow) return;
            arguments();
            const Arrays Ag = global_arrays<G>(p, u);
            unsigned long long* kc = p.key_c + (long long)u * p.c_stride;
            uint8_t* flc = p.flag_c + (long long)u * p.c_stride;
            if (tid == 0) {
                S.far[0] = 0;
                S.far[1] = 1;      // (the general path shifts by the largest logit)
            }
            LevelState<G> stc;
            const int lin = score_level<G>(p, L, Ag, S, u, p.n_coarse, false, true, p.coarse_budget, false, true, qv, kc, flc, stc);
            if (tid == 0) p.key_mode[2 * u] = lin;
            coarse_candidates<G>(p, Ag, L.A.ids, S, sc, u, n_f, n_terms);
            emit_coarse_terms<G>(p, Ag, u);
            leave_behind<G>(Ag, S, p.n_coarse, stc);
        }
        // the fine level reads the candidate list: from LDS, or back from global memory where it is long
        if (coarse_fast && n_f <= lds_cap) phase_sync<true>();
        else __syncthreads();
    }
    if (shadow) {
        if (n_f <= lds_cap) touch_rows(p, two ? L.A.ids : nullptr, u, n_f);
        return;
    }
    // (the coarse level's centroid terms are written while the fine level's rows travel)
    const auto coarse_terms = [&] {
        if (!two) arguments();
        if (two && coarse_fast && p.use_mp) fast_terms<G>(p, fc, slot_c, p.n_coarse, p.fcap, u);
    };
    if (n_f <= lds_cap) {
        FastLevel<G> ff_state;
        LevelTables fine = first;
        if (two) {
            const long long t = (long long)u * tab_rows;
            fine = LevelTables{Kc + t * kHeadDim, N + t, p.fstart + (long long)u * p.fstart_stride};
        }
        const int lin = fast_level<G, kHelped>(p, L, S, fine, n_f, u, two, false, two, !two, qv, false,
                                      kHelped && coarse_fast && S.early ? p.early + (long long)u * p.early_stride * (8 * GH) : nullptr, ff_state, coarse_terms);
        if (tid == 0) p.key_mode[2 * u + 1] = lin;
        fast_epilogue<G>(p, L, S, sc, ff_state, u, n_f, two, n_terms);
    } else {
        coarse_terms();
        if (two && coarse_fast) {      // (the general path reads the sums over all waves)
            if (tid < G) {
                double b = 0.0;
                for (int w = 0; w < kWaves; ++w) b += S.bw[w][tid];
                S.bs[tid] = b;
            }
            __syncthreads();
        }
        const Arrays Ag = global_arrays<G>(p, u);
        unsigned long long* kf = p.key_f + (long long)u * p.f_stride;
        uint8_t* ff = p.flag_f + (long long)u * p.f_stride;
        LevelState<G> stf;
        const int lin = score_level<G>(p, L, Ag, S, u, n_f, two, false, p.key_budget, two, !two, qv, kf, ff, stf);
        if (tid == 0) p.key_mode[2 * u + 1] = lin;
        fine_epilogue<G>(p, Ag, S, sc, u, n_f, two, n_terms);
    }
    // (whether or not they were waited for: when the last of them is done the count is zero again)
    if (kHelped && tid == 0) __hip_atomic_fetch_add(p.early_done + u, -helpers, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (appends)
        reinterpret_cast<uint4*>(p.app_dst[tid >> 4])[((long long)u * p.app_dst_rows + p.app_row) * 16 + (tid & 15)] = app;
}

}  // namespace

size_t score_smem_bytes(int G, int lds_cap)
{
    const size_t GH = (size_t)(G + 3) / 4;
    return align16(sizeof(Scratch)) + GH * 512 * 8 + (size_t)kHistBuckets * 8 + (size_t)kListCap * 16 +
           (size_t)lds_cap * (8 + 3 * 4) + 32;
}

template <int G, bool kHelped>
static hipError_t launch_score_g(const ScoreParams& p, int copies, hipStream_t s)
{
    static size_t configured = 48 * 1024;
    const size_t smem = score_smem_bytes(G, p.lds_cap);
    if (smem > configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&score_select_kernel<G, kHelped>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        configured = smem;
    }
    const bool two = p.levels == 2;
    hipLaunchKernelGGL((score_select_kernel<G, kHelped>), dim3(p.U * copies), dim3(kThreads), smem, s, p.q, p.Kc, p.N,
                       two ? p.cstart : p.fstart, p.U, (int)p.tab_rows, two ? p.fcap : 0, two ? p.n_coarse : p.n_fine,
                       (int)(two ? p.cstart_stride : p.fstart_stride), p.lds_cap, p.helpers, p.n_fine, p);
    return hipGetLastError();
}

hipError_t launch_score_select(const ScoreParams& p, int n_compute_units, bool helpers_run, hipStream_t s)
{
    // a shadow workgroup per unit where the chip has compute units to spare and the second workgroup
    // of unit u (block u + U) lands on the same L2 slice as the first (blocks go round the 8 slices)
    const bool helped = p.levels == 2 && p.helpers > 0;
    const int copies = helped ? 1 + (helpers_run ? p.helpers : 0) : (p.U % 8 == 0 && 2 * p.U <= n_compute_units) ? 2 : 1;
    switch (p.G) {
        case 1: return helped ? launch_score_g<1, true>(p, copies, s) : launch_score_g<1, false>(p, copies, s);
        case 2: return helped ? launch_score_g<2, true>(p, copies, s) : launch_score_g<2, false>(p, copies, s);
        case 3: return helped ? launch_score_g<3, true>(p, copies, s) : launch_score_g<3, false>(p, copies, s);
        case 4: return helped ? launch_score_g<4, true>(p, copies, s) : launch_score_g<4, false>(p, copies, s);
        case 5: return helped ? launch_score_g<5, true>(p, copies, s) : launch_score_g<5, false>(p, copies, s);
        case 6: return helped ? launch_score_g<6, true>(p, copies, s) : launch_score_g<6, false>(p, copies, s);
        case 7: return helped ? launch_score_g<7, true>(p, copies, s) : launch_score_g<7, false>(p, copies, s);
        case 8: return helped ? launch_score_g<8, true>(p, copies, s) : launch_score_g<8, false>(p, copies, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mp
