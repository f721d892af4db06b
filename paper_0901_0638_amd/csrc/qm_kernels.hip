/*
 * qm_kernels.hip -- streaming elementwise kernels for gfx950.
 *
 * One template covers every (kind, dtype, mode) of the normal quantile and
 * the exponential -> normal map, over wave tiles of 16-byte vectors
 * (qm_stream.hpp), the edge elements by the first workgroup.  The Student t
 * kernels (qm_student.hip) and the batch kernel (qm_batch.hip) reuse the
 * same walk and per-element functions.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "qm_device.hpp"
#include "qm_hybrid.hpp"
#include "qm_internal.h"

namespace qm {

template <typename T, int UNROLL, class Op>
__global__ __launch_bounds__(256) void k_map(Span<T> s)
{
    const uint32_t lane = wave_lane();
    const typename MapOf<T, Op>::type map{};
    Walk<T, UNROLL> w;
    w.begin(s, wave_uniform(blockIdx.x * 4ull + (threadIdx.x >> 6)), gridDim.x * 4ull, lane);
    w.run(s, lane, map);
    if (blockIdx.x == 0) run_edges(s, map);
}

/* The hybrid quantile over a memory stream (see qm_hybrid.hpp). */
template <typename T, int UNROLL, class H>
__global__ __launch_bounds__(256) void k_hybrid(Span<T> s)
{
    __shared__ T outer_buf[4][64 * Walk<T, UNROLL>::K];
    const uint32_t lane = wave_lane();
    const HybridMap<T, H> map = {outer_buf[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)], lane};
    Walk<T, UNROLL> w;
    w.begin(s, wave_uniform(blockIdx.x * 4ull + (threadIdx.x >> 6)), gridDim.x * 4ull, lane);
    w.run(s, lane, map);
    if (blockIdx.x == 0) run_edges(s, map);
}

template <typename T, class Op>
static hipError_t launch_op(const void* in, void* out, uint64_t n, hipStream_t s, const LaunchShape& shape)
{
    typedef typename HybridOf<Op>::type H;
    const bool gather = shape.compact && !std::is_void<H>::value;
    constexpr bool light = std::is_same<Op, OpE64Paper>::value || std::is_same<Op, OpNQ32Paper>::value ||
                           std::is_same<Op, OpNQ32Plain>::value;
    const bool f64 = sizeof(T) == 8;
    const KernelShape ks = gather ? shape.hybrid[f64] : light ? shape.light[f64] : f64 ? shape.stream : shape.stream32;
    const Span<T> a = make_span(static_cast<const T*>(in), static_cast<T*>(out), n);
    const int u = launch_unroll(a.nvec, ks, shape.cus);
    const dim3 grid(launch_blocks(a.nvec, u, ks)), block(256);
    with_unroll(u, [&](auto U) {
        if constexpr (!std::is_void<H>::value) {
            if (gather) {
                hipLaunchKernelGGL((k_hybrid<T, decltype(U)::value, H>), grid, block, 0, s, a);
                return;
            }
        }
        hipLaunchKernelGGL((k_map<T, decltype(U)::value, Op>), grid, block, 0, s, a);
    });
    return hipGetLastError();
}

hipError_t launch_elementwise(int kind, int dtype, int mode, const void* in, void* out, uint64_t n,
                              hipStream_t s, const LaunchShape& shape)
{
    if (kind == QM_NORMAL_QUANTILE) {
        if (dtype == QM_F64 && mode == QM_PLAIN) return launch_op<double, OpNQ64Plain>(in, out, n, s, shape);
        if (dtype == QM_F64 && mode == QM_PAPER) return launch_op<double, OpNQ64Paper>(in, out, n, s, shape);
        if (dtype == QM_F64 && mode == QM_PAPER_T2) return launch_op<double, OpNQ64PaperT2>(in, out, n, s, shape);
        if (dtype == QM_F32 && mode == QM_F32_REFINE) return launch_op<float, OpNQ32Refine>(in, out, n, s, shape);
        if (dtype == QM_F32 && mode == QM_PAPER) return launch_op<float, OpNQ32Paper>(in, out, n, s, shape);
        if (dtype == QM_F32 && mode == QM_PLAIN) return launch_op<float, OpNQ32Plain>(in, out, n, s, shape);
    } else if (kind == QM_EXP_TO_NORMAL) {
        if (dtype == QM_F64 && mode == QM_PLAIN) return launch_op<double, OpE64Plain>(in, out, n, s, shape);
        if (dtype == QM_F64 && mode == QM_PAPER) return launch_op<double, OpE64Paper>(in, out, n, s, shape);
        if (dtype == QM_F32 && mode == QM_F32_REFINE) return launch_op<float, OpE32Refine>(in, out, n, s, shape);
        if (dtype == QM_F32 && mode == QM_PLAIN) return launch_op<float, OpE32Plain>(in, out, n, s, shape);
    }
    return hipErrorInvalidValue;
}

}  // namespace qm
