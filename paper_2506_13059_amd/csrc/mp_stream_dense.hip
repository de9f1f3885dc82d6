// Dense attention on the matrix cores, for gfx950 (mp_stream.hip has the scheme): the rows of one source in order.  All that a wave needs
// are scalars of the launch, in registers when it starts, so its query and first rows are asked for at once; a launch over short contexts
// is little more than that chain (8 units x 4096 rows, 4 heads, workgroups of eight waves, of 20.9k cycles 1.9k went to the arguments: call
// 12.6 -> 11.8 us).
#include "mp_stream_tiles.h"

namespace mp {

namespace {

template <int G, int kWaves>
__global__ __launch_bounds__(64 * kWaves, 2) void value_dense_kernel(const uint16_t* q, const uint16_t* K, const uint16_t* V, float* partials,
                                                                    int n, int n_units, int chunk_rows, int chunks_per_unit, float scale_log2e)
{
    extern __shared__ __align__(256) unsigned char ring_lds[];
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t ring = (uint32_t)(uintptr_t)(lds_byte*)ring_lds + (uint32_t)(wave * kRing);
    const int chunk = blockIdx.x / n_units, u = blockIdx.x - chunk * n_units;
    const int begin = chunk * chunk_rows, end = min(begin + chunk_rows, n);
    const int wave_rows = (chunk_rows / kWaves + kTile - 1) / kTile * kTile;
    const int w0 = begin + wave * wave_rows, w1 = min(w0 + wave_rows, end);
    float* part = partials + ((long long)u * chunks_per_unit + chunk) * G * kPartStride;
    if (begin >= end) {
        if (tid < G) {
            part[tid * kPartStride + 0] = -INFINITY;
            part[tid * kPartStride + 1] = 0.f;
        }
        return;
    }
    RowSource S{};
    S.K = K;
    S.V = V;
    S.unit_rows = n;
    ValuePassParams p{};
    p.q = q;
    p.scale_log2e = scale_log2e;
    StreamState<G> st;
    clear_state(st);
    if (w0 < w1) stream_tiles<G, false, false>(st, S, p, u, w0, w1, ring, 0u, [] {});
    combine_waves<G, kWaves>(st, reinterpret_cast<float*>(ring_lds), part);
}

template <int G, int kWaves>
hipError_t launch_dense_w(const ValuePassParams& p, unsigned blocks, hipStream_t s)
{
    static bool configured = false;
    constexpr size_t smem = kWaves * kRing;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&value_dense_kernel<G, kWaves>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    const RowSource& S = p.src[0];
    hipLaunchKernelGGL((value_dense_kernel<G, kWaves>), dim3(blocks), dim3(64 * kWaves), smem, s, p.q, S.K, S.V, p.partials, S.count_max, p.n_units,
                       S.chunk_rows, p.chunks_per_unit, p.scale_log2e);
    return hipGetLastError();
}

// Four waves a workgroup, or eight where the launch leaves half of the compute units idle and a wave's share is a long chain of tiles
// all the same: 8 units x 4096 rows, 4 / 8 heads: 13.4 / 15.3 us with four waves, 12.8 / 14.7 with eight (before the scalars).
template <int G>
hipError_t launch_dense_g(const ValuePassParams& p, hipStream_t s)
{
    const long long blocks = (long long)p.n_units * p.chunks_per_unit;
    if (blocks <= 0) return hipSuccess;
    const bool eight = blocks <= 128 && p.src[0].chunk_rows >= 512;
    return eight ? launch_dense_w<G, 8>(p, (unsigned)blocks, s) : launch_dense_w<G, 4>(p, (unsigned)blocks, s);
}

}  // namespace

hipError_t launch_value_dense(const ValuePassParams& p, int G, hipStream_t s)
{
    const RowSource& S = p.src[0];
    if (p.n_sources != 1 || S.rows || S.scores || S.count_dev || S.row0 != 0 || S.chunk0 != 0 || S.unit_rows != S.count_max) return hipErrorInvalidValue;
    switch (G) {
        case 1: return launch_dense_g<1>(p, s);
        case 2: return launch_dense_g<2>(p, s);
        case 3: return launch_dense_g<3>(p, s);
        case 4: return launch_dense_g<4>(p, s);
        case 5: return launch_dense_g<5>(p, s);
        case 6: return launch_dense_g<6>(p, s);
        case 7: return launch_dense_g<7>(p, s);
        case 8: return launch_dense_g<8>(p, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mp
