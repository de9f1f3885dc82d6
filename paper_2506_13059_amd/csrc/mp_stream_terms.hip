// Value pass of a decode step over bf16 rows whose centroid terms have a wave of their own, for gfx950 (mp_stream.hip has the scheme).
//
// A launch over a short selection is a chain of trips to memory, and the centroid terms that ride along with the selected keys were
// one more link of it: their row numbers and rows come after a wave's own.  Here a fifth wave of the workgroup takes the workgroup's
// terms while four stream its keys; its ring holds logits in the place of keys, so that two workgroups still fit a compute unit.
// What the first requests need are scalars of the launch, in registers when a wave starts: the row numbers and the
// counts do not wait for the other arguments.
//
// Cycles of a workgroup before, 8 units x 4096 keys of 4 heads (17.3k in all): arguments and counts 2.5k, row numbers 0.9k, first keys 3.2k, their
// values 2.0k, the rest of the keys 2.3k, the terms 3.0k, the combination 2.1k.  Whole step 24.6 -> 23.5 us, 32 units of 5 heads 37.6 ->
// 36.5, 128 units x 8192 keys 120.3 -> 118.5 (with rows of 132 words in the combination, which the other kernels have, too).
#include "mp_stream_tiles.h"

namespace mp {

namespace {

constexpr int kKeyWaves = 4;
constexpr int kTermsBytes = kScoredRing + 8 * kStrip;

// rows, n_rows, rows_stride, chunk0, chunk_rows: the selected keys' source, the launch's last; n_terms: number of the terms, src[0].
template <int G>
__global__ __launch_bounds__(64 * (kKeyWaves + 1), 2) void value_terms_kernel(const int32_t* rows, const int32_t* n_rows, const int32_t* n_terms,
                                                                             int rows_stride, int n_units, int chunk0, int chunk_rows,
                                                                             const ValuePassParams p)
{
    extern __shared__ __align__(256) unsigned char ring_lds[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)ring_lds;
    const uint32_t ring = lds0 + (uint32_t)(wave * kRing);
    const uint32_t strips = lds0 + (uint32_t)(wave < kKeyWaves ? kKeyWaves * kRing + kScoredRing + wave * 8 * kStrip : kKeyWaves * (kRing + 8 * kStrip) + kScoredRing);
    const int chunk = blockIdx.x / n_units, u = blockIdx.x - chunk * n_units;
    const bool keys = chunk >= chunk0;      // (the others have rows of the tail)
    typedef const __attribute__((address_space(4))) int32_t constant_int;
    int counted = 0, terms = 0;
    if (keys) {
        counted = ((constant_int*)n_rows)[u];
        terms = ((constant_int*)n_terms)[u];
        if (wave < kKeyWaves) {
            const int first = (chunk - chunk0) * chunk_rows + wave * ((chunk_rows / kKeyWaves + kTile - 1) / kTile * kTile);
            load_to_lds<4, false>(rows + (long long)u * rows_stride + min(first + (tid & 63), rows_stride - 1), strips);
        }
    }
    touch_arguments(p);
    asm volatile("" ::"s"(counted), "s"(terms));
    const RowSource& S = p.src[keys ? p.n_sources - 1 : 1];
    const RowSource& T = p.src[0];
    const int begin = (chunk - S.chunk0) * S.chunk_rows;
    const int end = min(begin + S.chunk_rows, keys ? min(counted, S.count_max) : S.count_max);
    const int wave_rows = (S.chunk_rows / kKeyWaves + kTile - 1) / kTile * kTile;
    const int w0 = begin + wave * wave_rows, w1 = min(w0 + wave_rows, end);
    int g0 = 0, g1 = 0;
    if (keys) {
        const long long n = min(terms, T.count_max), k = chunk - chunk0;
        g0 = (int)(n * k / S.n_chunks);
        g1 = (int)(n * (k + 1) / S.n_chunks);
    }
    float* part = p.partials + ((long long)u * p.chunks_per_unit + chunk) * G * kPartStride;
    if (begin >= end && g0 >= g1) {
        nothing_on_its_way();
        if (tid < G) {
            part[tid * kPartStride + 0] = -INFINITY;
            part[tid * kPartStride + 1] = 0.f;
        }
        return;
    }
    // the rows of this wave
    const bool of_terms = wave == kKeyWaves;
    const int a = of_terms ? g0 : w0, b = of_terms ? g1 : w1;
    if (of_terms && a < b) fetch_strip(T.rows, T, u, a, strips);
    if (a >= b) nothing_on_its_way();       // (its first row numbers are in place before the space is used)
    StreamState<G> st;
    clear_state(st);
    if (a < b) {
        if (of_terms) stream_tiles<G, true, true>(st, T, p, u, a, b, ring, strips, [] {});
        else if (keys) stream_tiles<G, false, true>(st, S, p, u, a, b, ring, strips, [] {});
        else stream_tiles<G, false, false>(st, S, p, u, a, b, ring, strips, [] {});
    }
    combine_waves<G, kKeyWaves + 1>(st, reinterpret_cast<float*>(ring_lds), part);
}

template <int G>
hipError_t launch_terms_g(const ValuePassParams& p, hipStream_t s)
{
    static bool configured = false;
    constexpr size_t smem = kKeyWaves * (kRing + 8 * kStrip) + kTermsBytes;
    static_assert(2 * smem <= 160 * 1024, "two workgroups a compute unit");
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&value_terms_kernel<G>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    const RowSource& S = p.src[p.n_sources - 1];
    hipLaunchKernelGGL((value_terms_kernel<G>), dim3((unsigned)((long long)p.n_units * p.chunks_per_unit)), dim3(64 * (kKeyWaves + 1)), smem, s, S.rows,
                       S.count_dev, p.src[0].count_dev, (int)S.rows_stride, p.n_units, S.chunk0, S.chunk_rows, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_value_terms(const ValuePassParams& p, int G, hipStream_t s)
{
    // src[0] the terms, perhaps a tail, the selected keys
    const RowSource &T = p.src[0], &S = p.src[p.n_sources - 1];
    if (p.n_sources < 2 || p.n_sources > 3 || !S.guest || !S.rows || !S.count_dev || S.row0 != 0 || !T.scores || !T.count_dev || T.n_chunks != 0 ||
        S.rows_stride > 0x7fffffff || (p.n_sources == 3 && (p.src[1].rows || p.src[1].count_dev || p.src[1].row0 != 0)))
        return hipErrorInvalidValue;
    switch (G) {
        case 1: return launch_terms_g<1>(p, s);
        case 2: return launch_terms_g<2>(p, s);
        case 3: return launch_terms_g<3>(p, s);
        case 4: return launch_terms_g<4>(p, s);
        case 5: return launch_terms_g<5>(p, s);
        case 6: return launch_terms_g<6>(p, s);
        case 7: return launch_terms_g<7>(p, s);
        case 8: return launch_terms_g<8>(p, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mp
