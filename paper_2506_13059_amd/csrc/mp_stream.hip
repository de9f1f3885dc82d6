// Value pass on the matrix cores, for gfx950: the counterpart of value_pass_kernel (mp_value.hip) for groups of
// query heads whose arithmetic a vector pipe cannot do at the rate the rows arrive.  The kernel here serves decode steps over bf16
// rows whose centroid terms ride along with the selected keys or are left out, and steps that select no keys; the others and
// dense calls have kernels of the same scheme (mp_stream_terms.hip, mp_stream_dense.hip, mp_stream8.hip).
//
// A wave streams tiles of 16 rows.  Rows go from global memory straight to LDS (global_load_lds, 16 bytes a lane,
// four whole rows an instruction), into a ring of two tiles per wave, so that three of the four 4 KiB pieces are on
// their way while one is used and no registers are held for them.  Per tile:
//   S = K Q^T      four v_mfma_f32_16x16x32_bf16 (A = 16 key rows, B = up to 16 columns of queries); lane (g, c)
//                  receives rows 4g .. 4g+3 of column c
//   P = 2^(S - m)  online softmax in fp32, one column (head) per lane, rescaling only when a maximum moves
//   O += P V       eight v_mfma_f32_16x16x16_bf16 (A = P exactly as it lies in the registers, B = V read from LDS
//                  with the transposing read)
// The matrix cores take bf16, the probabilities are fp32: each is split exactly into three bf16 values (8 + 8 + 8
// significant bits, by truncation), and the 16 columns of the product hold them side by side: column part * G + h.
// Where three parts of G heads do not fit 16 columns (G > 5) the third parts take a second set of products.  The
// sum of the parts' products is the fp32 product sum; nothing is rounded to 16 bits.
// Infinite values come out as the products of the fp32 probabilities would have them: see part_floor, and the rows past
// the end of a wave's share are zeros by the time their probability of zero meets them.
//
// What bounds it is the memory system: about 100 vector instructions a tile against 420 of the vector-ALU kernel (60 %
// of a SIMD's issue slots at the dense rate with 4 heads, more than there are with 8).  Measured on the benchmark's
// 8 GiB cache, dense, which this kernel served then (value_dense_kernel has the same tiles), 1 / 4 / 5 / 6 / 8 heads: vector ALU
// 1259 / 1345 / 1367 / 1615 / 1763 us, here with the same chunks 1263 / 1341 / 1358 / 1382 / 1409 us, with one workgroup per
// compute unit (see plan_streams in mp_plan.h) 1230 / 1228 / - / - / 1233 us = 7.0 TB/s; 64 units x 60013 rows, 8 heads: the
// call 505 -> 301 to 306 us, 294 of them the kernel; 8 units x 32768, 4 heads: 40.8 -> 26.0 us.
#include "mp_stream_tiles.h"

namespace mp {

namespace {

template <int G, int kWaves>
__global__ __launch_bounds__(64 * kWaves, 2) void value_stream_kernel(const ValuePassParams p)
{
    extern __shared__ __align__(256) unsigned char ring_lds[];
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)ring_lds;
    const uint32_t ring = lds0 + (uint32_t)(wave * kRing), strips = lds0 + (uint32_t)(kWaves * kRing + wave * kStripBytes);
    const uint32_t guest_strip = strips + 8 * kStrip;
    touch_arguments(p);
    const StreamShare w = stream_share<kWaves>(p, [&](const RowSource& S, int u, int first) { fetch_strip(S.rows, S, u, first, strips); });
    const RowSource& S = p.src[w.source];
    const int u = w.u;
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
        if (S.scores) stream_tiles<G, true, true>(st, S, p, u, w.w0, w.w1, ring, strips, guest);
        else if (S.rows) stream_tiles<G, false, true>(st, S, p, u, w.w0, w.w1, ring, strips, guest);
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
hipError_t launch_stream_g(const ValuePassParams& p, hipStream_t s)
{
    const long long blocks = (long long)p.n_units * p.chunks_per_unit;
    if (blocks <= 0) return hipSuccess;
    constexpr int kWaves = 4;
    static bool configured = false;
    constexpr size_t smem = kWaves * (kRing + kStripBytes);
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&value_stream_kernel<G, kWaves>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL((value_stream_kernel<G, kWaves>), dim3((unsigned)blocks), dim3(64 * kWaves), smem, s, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_value_stream(const ValuePassParams& p, int G, hipStream_t s)
{
    switch (G) {
        case 1: return launch_stream_g<1>(p, s);
        case 2: return launch_stream_g<2>(p, s);
        case 3: return launch_stream_g<3>(p, s);
        case 4: return launch_stream_g<4>(p, s);
        case 5: return launch_stream_g<5>(p, s);
        case 6: return launch_stream_g<6>(p, s);
        case 7: return launch_stream_g<7>(p, s);
        case 8: return launch_stream_g<8>(p, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mp
