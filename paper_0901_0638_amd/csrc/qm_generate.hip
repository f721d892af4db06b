/*
 * qm_generate.hip -- fused generation and transform: the open uniforms of a
 * Philox4x32-10 stream (qm_philox.hpp) are drawn in registers and mapped
 * (identity, or the normal quantile in any of its forms) before the only
 * memory access, the 16-byte store of the results -- 8 bytes per FP64
 * sample instead of the 16 of a separate generate-then-transform pass
 * (the reuse of uniform streams the paper's maps are built for).
 *
 * Each lane takes whole Philox blocks: one block is one 16-byte vector of
 * outputs (two FP64 or four FP32 samples).  The hybrid quantiles gather
 * their outer elements across the wave exactly as the streaming kernel does
 * (hybrid_eval), so every output is bitwise the one qm_normal_quantile gives
 * for the same uniform.  Outputs before the first block boundary and after
 * the last whole block (fewer than two blocks' worth) are done one element
 * at a time by the same per-element functions.
 *
 * The 16-byte stores need only the element's alignment (gfx950 takes a
 * dwordx4 access at any dword), so every sub-range of a stream and every
 * output address goes through whole blocks.  A stream index and an address
 * that disagree modulo 16 bytes used to draw each element's block afresh,
 * twice the Philox work in FP64 and four times in FP32, and to vote instead
 * of gather: 2^24 FP64 Student t samples from an odd element took 141 us on
 * MI355X, and 75 here; FP32 quantiles from one 71, and 26 here.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>
#include <type_traits>

#include "qm_hybrid.hpp"
#include "qm_hyp_device.hpp"
#include "qm_internal.h"
#include "qm_philox.hpp"
#include "qm_stream.hpp"
#include "qm_student_device.hpp"

namespace qm {

template <typename T>
struct GenArgs {
    T* out;
    uint32_t k0, k1;
    uint64_t first;       /* stream index of out[0] */
    uint64_t head;        /* out[0, head): before the first block boundary */
    uint64_t nvec;        /* whole blocks from out[head] on */
    uint64_t tail_begin;  /* out[tail_begin, n): after the last whole block */
    uint64_t n;
};

/* the NV uniforms of block b */
__device__ __forceinline__ void block_uniforms(uint64_t b, uint32_t k0, uint32_t k1, double (&u)[2])
{
    PhiloxWords w = philox4x32_10(b, k0, k1);
    u[0] = open_u53(w.w[0], w.w[1]);
    u[1] = open_u53(w.w[2], w.w[3]);
}
__device__ __forceinline__ void block_uniforms(uint64_t b, uint32_t k0, uint32_t k1, float (&u)[4])
{
    PhiloxWords w = philox4x32_10(b, k0, k1);
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = open_u23(w.w[j]);
}

/* H: the per-element map (Op), or with GATHER the hybrid (HybridNQ64/32). */
template <typename T, int UNROLL, class H, bool GATHER>
__global__ __launch_bounds__(256) void k_generate(GenArgs<T> a)
{
    typedef typename vec16any<T>::type V;
    constexpr int NV = vec16<T>::n;
    constexpr int K = NV * UNROLL;
    const uint32_t lane = wave_lane();
    __shared__ T outer_buf[GATHER ? 4 : 1][GATHER ? 64 * K : 1];
    T* buf = outer_buf[GATHER ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0];
    V* vout = reinterpret_cast<V*>(a.out + a.head);
    const uint64_t block0 = (a.first + a.head) / NV;
    /* wave-contiguous tiles of 64 UNROLL vectors, dealt out to the waves
       in turn; whole waves iterate together, as the gather needs.  Whole
       tiles store without bound tests; in the one partial last tile the
       blocks past the end are drawn but not stored. */
    constexpr uint64_t TILE = 64ull * UNROLL;
    const uint64_t step = (uint64_t)gridDim.x * 4 * TILE;
    auto tile = [&](uint64_t t, auto whole) {
        const uint64_t i = t + lane;
        T u[K], w[K];
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            T b[NV];
            block_uniforms(block0 + i + 64 * k, a.k0, a.k1, b);
#pragma unroll
            for (int j = 0; j < NV; ++j) u[NV * k + j] = b[j];
        }
        if constexpr (GATHER) {
            hybrid_eval<T, K, H>(u, w, buf, lane);
        } else {
            H op;
#pragma unroll
            for (int k = 0; k < K; ++k) w[k] = op(u[k]);
        }
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            uint64_t idx = i + 64 * k;
            V y;
#pragma unroll
            for (int j = 0; j < NV; ++j) y[j] = w[NV * k + j];
            if (decltype(whole)::value || idx < a.nvec) __builtin_nontemporal_store(y, vout + idx);
        }
    };
    uint64_t t = wave_uniform(((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * TILE);
    for (; t + TILE <= a.nvec; t += step) tile(t, std::true_type());
    if (t < a.nvec) tile(t, std::false_type());
    if (blockIdx.x == 0) {
        uint64_t extra = a.head + (a.n - a.tail_begin);
        for (uint64_t e = threadIdx.x; e < extra; e += blockDim.x) {
            uint64_t idx = e < a.head ? e : a.tail_begin + (e - a.head);
            T u = stream_uniform<T>(a.first + idx, a.k0, a.k1);
            if constexpr (GATHER) a.out[idx] = H::whole(u);
            else a.out[idx] = H()(u);
        }
    }
}

/* The blocks of a generate launch: head, whole blocks, tail. */
template <typename T>
static void gen_geometry(GenArgs<T>& a)
{
    constexpr int NV = vec16<T>::n;
    a.head = (NV - a.first % NV) % NV;
    if (a.head > a.n) a.head = a.n;
    a.nvec = (a.n - a.head) / NV;
    a.tail_begin = a.head + a.nvec * NV;
}

template <typename T, class H, bool GATHER>
static hipError_t launch_gen(GenArgs<T> a, hipStream_t s, const LaunchShape& shape)
{
    const KernelShape ks = (std::is_same<H, OpCopy<T>>::value ? shape.uniform : shape.generate)[sizeof(T) == 8];
    gen_geometry(a);
    const int u = launch_unroll(a.nvec, ks, shape.cus);
    with_unroll(u, [&](auto U) {
        hipLaunchKernelGGL((k_generate<T, decltype(U)::value, H, GATHER>), dim3(launch_blocks(a.nvec, u, ks)), dim3(256),
                           0, s, a);
    });
    return hipGetLastError();
}

hipError_t launch_generate(int kind, int dtype, int mode, uint32_t seed, uint32_t stream, uint64_t first,
                           void* out, uint64_t n, hipStream_t s, const LaunchShape& shape)
{
    if (dtype == QM_F64) {
        GenArgs<double> a{};
        a.out = static_cast<double*>(out);
        a.k0 = seed;
        a.k1 = stream;
        a.first = first;
        a.n = n;
        if (kind == QM_UNIFORM && mode == QM_PLAIN) return launch_gen<double, OpCopy<double>, false>(a, s, shape);
        if (kind == QM_NORMAL_QUANTILE && mode == QM_PLAIN) {
            if (shape.compact) return launch_gen<double, HybridNQ64, true>(a, s, shape);
            return launch_gen<double, OpNQ64Plain, false>(a, s, shape);
        }
        if (kind == QM_NORMAL_QUANTILE && mode == QM_PAPER) return launch_gen<double, OpNQ64Paper, false>(a, s, shape);
    } else if (dtype == QM_F32) {
        GenArgs<float> a{};
        a.out = static_cast<float*>(out);
        a.k0 = seed;
        a.k1 = stream;
        a.first = first;
        a.n = n;
        if (kind == QM_UNIFORM && mode == QM_PLAIN) return launch_gen<float, OpCopy<float>, false>(a, s, shape);
        if (kind == QM_NORMAL_QUANTILE && mode == QM_F32_REFINE) {
            if (shape.compact) return launch_gen<float, HybridNQ32, true>(a, s, shape);
            return launch_gen<float, OpNQ32Refine, false>(a, s, shape);
        }
        if (kind == QM_NORMAL_QUANTILE && mode == QM_PAPER) return launch_gen<float, OpNQ32Paper, false>(a, s, shape);
        if (kind == QM_NORMAL_QUANTILE && mode == QM_PLAIN) return launch_gen<float, OpNQ32Plain, false>(a, s, shape);
    }
    return hipErrorInvalidValue;
}

StudentParams make_params(const TTableHeader& h, const TCells& c, const double* d_rows);


/* Fused uniform -> normal -> Student t.  The quantile stage is the one of
   k_generate (H, gathered per wave with GATHER); each normal then goes
   through student_eval from the LDS table, as in k_student. */
template <typename T, int UNROLL, class H, bool GATHER, int DEG>
__global__ __launch_bounds__(256) void k_generate_t(GenArgs<T> a, StudentParams P)
{
    extern __shared__ __attribute__((aligned(16))) double lds_gt[];
    stage_table(lds_gt, P.gcoef, P);
    __syncthreads();
    typedef typename vec16any<T>::type V;
    constexpr int NV = vec16<T>::n;
    constexpr int K = NV * UNROLL;
    const StudentMap<T, DEG> tmap = {lds_gt, P};
    const uint32_t lane = wave_lane();
    __shared__ T outer_buf[GATHER ? 4 : 1][GATHER ? 64 * K : 1];
    T* buf = outer_buf[GATHER ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0];
    V* vout = reinterpret_cast<V*>(a.out + a.head);
    const uint64_t block0 = (a.first + a.head) / NV;
    /* wave-contiguous tiles of 64 UNROLL vectors, as k_generate: whole
       tiles store without bound tests, the one partial last tile draws
       its blocks past the end but does not store them */
    constexpr uint64_t TILE = 64ull * UNROLL;
    const uint64_t step = (uint64_t)gridDim.x * 4 * TILE;
    auto tile = [&](uint64_t t, auto whole) {
        const uint64_t i = t + lane;
        T u[K], w[K];
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            T b[NV];
            block_uniforms(block0 + i + 64 * k, a.k0, a.k1, b);
#pragma unroll
            for (int j = 0; j < NV; ++j) u[NV * k + j] = b[j];
        }
        if constexpr (GATHER) {
            hybrid_eval<T, K, H>(u, w, buf, lane);
        } else {
            H op;
#pragma unroll
            for (int k = 0; k < K; ++k) w[k] = op(u[k]);
        }
        tmap.tile(w, u);
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            uint64_t idx = i + 64 * k;
            V y;
#pragma unroll
            for (int j = 0; j < NV; ++j) y[j] = u[NV * k + j];
            if (decltype(whole)::value || idx < a.nvec) __builtin_nontemporal_store(y, vout + idx);
        }
    };
    uint64_t t = wave_uniform(((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * TILE);
    for (; t + TILE <= a.nvec; t += step) tile(t, std::true_type());
    if (t < a.nvec) tile(t, std::false_type());
    if (blockIdx.x == 0) {
        uint64_t extra = a.head + (a.n - a.tail_begin);
        for (uint64_t e = threadIdx.x; e < extra; e += blockDim.x) {
            uint64_t idx = e < a.head ? e : a.tail_begin + (e - a.head);
            T u = stream_uniform<T>(a.first + idx, a.k0, a.k1);
            T z;
            if constexpr (GATHER) z = H::whole(u);
            else z = H()(u);
            a.out[idx] = tmap.one(z);
        }
    }
}

/* The two-sided exponential base sample of an open uniform (Section 8.1),
   in FP64: one logarithm of the side's ratio, by the reduced atanh-series
   log of the quantile path (neg_log_unit; about an ulp, a third of the
   instructions of the library log).  The ratio is a product with the
   side's reciprocal mass, selected before one multiply: two IEEE divisions
   on diverged lanes had cost some 20 instructions per sample. */
struct HypBase {
    double p_minus, inv_p_minus, inv_p_plus, inv_rate_minus, inv_rate_plus;
    __device__ __forceinline__ double operator()(double u) const
    {
        /* u / p_minus < 1 < (1 - u) / p_plus on the left of the mode, the other
           way round on its right */
        const double ratio = __builtin_fmin(u * inv_p_minus, (1.0 - u) * inv_p_plus);
        /* u = 1 (an FP64 uniform of the top 53-bit value rounds to 1) is the
           base's right end, v = +inf (mapped to +inf): the logarithm of 0 is
           finite, and the infinity is added */
        const double l = neg_log_unit(ratio) + __hiloint2double(ratio > 0.0 ? 0 : 0x7ff00000, 0);
        return l * select_f64(u < p_minus, -inv_rate_minus, inv_rate_plus);
    }
};

/* The base's constants as the fused hyperbolic kernel takes them: p- and p+
   as exp of the table's log masses, their reciprocals, and the reciprocal
   rates 1/(alpha + beta) and 1/(alpha - beta), each one rounding. */
static void hyp_base_constants(const HypTableHeader& h, HypBase* B)
{
    B->p_minus = std::exp(h.log_p_minus);
    B->inv_p_minus = 1.0 / B->p_minus;
    B->inv_p_plus = 1.0 / std::exp(h.log_p_plus);
    B->inv_rate_minus = 1.0 / (h.alpha + h.beta);
    B->inv_rate_plus = 1.0 / (h.alpha - h.beta);
}

/* Fused uniform -> base sample -> hyperbolic: all K elements of a lane
   through the LDS cells, then one wave vote for the far ones (as
   k_hyperbolic). */
template <typename T, int UNROLL, int DEG>
__global__ __launch_bounds__(256) void k_generate_h(GenArgs<T> a, HypParams P, HypBase B)
{
    extern __shared__ __attribute__((aligned(16))) double lds_gh[];
    stage_hyp<DEG>(lds_gh, P);
    __syncthreads();
    typedef typename vec16any<T>::type V;
    constexpr int NV = vec16<T>::n;
    constexpr int K = NV * UNROLL;
    auto one = [&](T u) {
        const double v[1] = {B((double)u)};
        double q[1];
        hyp_abs_q<DEG, 1>(v, q, lds_gh, P);
        return (T)(P.mu + __builtin_copysign(q[0], v[0]));
    };
    V* vout = reinterpret_cast<V*>(a.out + a.head);
    const uint64_t block0 = (a.first + a.head) / NV;
    const uint32_t lane = wave_lane();
    /* wave-contiguous tiles, as k_generate (whole tiles unchecked, the
       partial last one checked) */
    constexpr uint64_t TILE = 64ull * UNROLL;
    const uint64_t step = (uint64_t)gridDim.x * 4 * TILE;
    auto tile = [&](uint64_t t, auto whole) {
        const uint64_t i = t + lane;
        double v[K], q[K];
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            T b[NV];
            /* blocks past the end are drawn but never stored */
            block_uniforms(block0 + i + 64 * k, a.k0, a.k1, b);
#pragma unroll
            for (int j = 0; j < NV; ++j) v[NV * k + j] = B((double)b[j]);
        }
        hyp_abs_q<DEG, K>(v, q, lds_gh, P);
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            uint64_t idx = i + 64 * k;
            V y;
#pragma unroll
            for (int j = 0; j < NV; ++j) y[j] = (T)(P.mu + __builtin_copysign(q[NV * k + j], v[NV * k + j]));
            if (decltype(whole)::value || idx < a.nvec) __builtin_nontemporal_store(y, vout + idx);
        }
    };
    uint64_t t = wave_uniform(((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * TILE);
    for (; t + TILE <= a.nvec; t += step) tile(t, std::true_type());
    if (t < a.nvec) tile(t, std::false_type());
    if (blockIdx.x == 0) {
        uint64_t extra = a.head + (a.n - a.tail_begin);
        for (uint64_t e = threadIdx.x; e < extra; e += blockDim.x) {
            uint64_t idx = e < a.head ? e : a.tail_begin + (e - a.head);
            a.out[idx] = one(stream_uniform<T>(a.first + idx, a.k0, a.k1));
        }
    }
}

template <typename T, class H, bool GATHER, int DEG>
static hipError_t launch_gen_t(GenArgs<T> a, const StudentParams& P, size_t lds, hipStream_t s, const KernelShape& ks,
                               int u)
{
    with_unroll(u, [&](auto U) {
        hipLaunchKernelGGL((k_generate_t<T, decltype(U)::value, H, GATHER, DEG>), dim3(launch_blocks(a.nvec, u, ks)),
                           dim3(256), lds, s, a, P);
    });
    return hipGetLastError();
}

/* LDS the gather buffer of a generate kernel takes (4 waves x 64 lanes x K) */
template <typename T>
static size_t gather_bytes(int unroll)
{
    return (size_t)4 * 64 * vec16<T>::n * unroll * sizeof(T);
}

constexpr size_t GEN_LDS_MAX = 65536;   /* static + dynamic LDS of a generate workgroup */

hipError_t launch_generate_student(int dtype, int mode, uint32_t seed, uint32_t stream, uint64_t first, void* out,
                                   uint64_t n, const TTableHeader* d_table, const TTableHeader& h, hipStream_t s,
                                   const LaunchShape& shape)
{
    if (h.identity) return launch_generate(QM_NORMAL_QUANTILE, dtype, mode, seed, stream, first, out, n, s, shape);
    const bool f64 = dtype == QM_F64 && mode == QM_PLAIN;
    if (!f64 && !(dtype == QM_F32 && mode == QM_F32_REFINE)) return hipErrorInvalidValue;
    const TCells& c = f64 ? h.f64 : h.f32;
    const StudentParams P = make_params(h, c, table_block(d_table) + c.coef_offset);
    const size_t lds = student_lds_bytes(P);
    const KernelShape ks = shape.generate_t[f64];
    if (lds > GEN_LDS_MAX) return hipErrorInvalidValue;
    auto launch = [&](auto a) {
        typedef typename std::remove_pointer<decltype(a.out)>::type T;
        a.out = static_cast<T*>(out);
        a.k0 = seed;
        a.k1 = stream;
        a.first = first;
        a.n = n;
        gen_geometry(a);
        const int u = launch_unroll(a.nvec, ks, shape.cus);
        /* the quantile stage gathers per wave when its buffer fits beside the
           table (bitwise the same results either way) */
        const bool gather = shape.compact && lds + gather_bytes<T>(u) <= GEN_LDS_MAX;
        if constexpr (std::is_same<T, double>::value) {
            if (c.degree == T_DEGREE_LOW) {
                if (gather) return launch_gen_t<T, HybridNQ64, true, T_DEGREE_LOW>(a, P, lds, s, ks, u);
                return launch_gen_t<T, OpNQ64Plain, false, T_DEGREE_LOW>(a, P, lds, s, ks, u);
            }
            if (gather) return launch_gen_t<T, HybridNQ64, true, T_DEGREE_HIGH>(a, P, lds, s, ks, u);
            return launch_gen_t<T, OpNQ64Plain, false, T_DEGREE_HIGH>(a, P, lds, s, ks, u);
        } else {
            if (gather) return launch_gen_t<T, HybridNQ32, true, T_DEGREE_F32>(a, P, lds, s, ks, u);
            return launch_gen_t<T, OpNQ32Refine, false, T_DEGREE_F32>(a, P, lds, s, ks, u);
        }
    };
    return f64 ? launch(GenArgs<double>{}) : launch(GenArgs<float>{});
}

template <typename T, int DEG>
static hipError_t launch_gen_h(GenArgs<T> a, const HypParams& P, const HypBase& B, size_t lds, hipStream_t s,
                               const LaunchShape& shape)
{
    const KernelShape ks = shape.generate_h[sizeof(T) == 8];
    gen_geometry(a);
    const int u = launch_unroll(a.nvec, ks, shape.cus);
    with_unroll(u, [&](auto U) {
        hipLaunchKernelGGL((k_generate_h<T, decltype(U)::value, DEG>), dim3(launch_blocks(a.nvec, u, ks)), dim3(256), lds,
                           s, a, P, B);
    });
    return hipGetLastError();
}

hipError_t launch_generate_hyperbolic(int dtype, int mode, uint32_t seed, uint32_t stream, uint64_t first, void* out,
                                      uint64_t n, const HypTableHeader* d_table, const HypTableHeader& h,
                                      uint64_t ncoef, double mu, hipStream_t s, const LaunchShape& shape)
{
    const bool f32 = dtype == QM_F32 && mode == QM_F32_REFINE;
    if (!f32 && !(dtype == QM_F64 && mode == QM_PLAIN)) return hipErrorInvalidValue;
    HypParams P;
    size_t lds = 0;
    if (!make_hyp_params(h, f32, d_table, ncoef, mu, &P, &lds)) return hipErrorInvalidValue;
    HypBase B;
    hyp_base_constants(h, &B);
    if (f32) {
        GenArgs<float> a{};
        a.out = static_cast<float*>(out);
        a.k0 = seed;
        a.k1 = stream;
        a.first = first;
        a.n = n;
        return launch_gen_h<float, HYP_DEGREE_F32>(a, P, B, lds, s, shape);
    }
    GenArgs<double> a{};
    a.out = static_cast<double*>(out);
    a.k0 = seed;
    a.k1 = stream;
    a.first = first;
    a.n = n;
    return launch_gen_h<double, HYP_DEGREE>(a, P, B, lds, s, shape);
}

}  // namespace qm
