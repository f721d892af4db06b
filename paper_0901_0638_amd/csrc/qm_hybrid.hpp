/*
 * qm_hybrid.hpp -- the per-element maps as kernel functors, and the
 * wave-level gather of the hybrid quantiles (shared by the streaming and the
 * generating kernels).
 */
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qm_device.hpp"
#include "qm_stream.hpp"

namespace qm {

struct OpNQ64Plain { __device__ double operator()(double u) const { return normal_quantile_f64<false>(u); } };
struct OpNQ64Paper { __device__ double operator()(double u) const { return normal_quantile_f64<true>(u); } };
struct OpNQ64PaperT2 { __device__ double operator()(double u) const { return normal_quantile_f64_t2(u); } };
struct OpE64Paper  { __device__ double operator()(double x) const { return exp_to_normal_f64_paper(x); } };
struct OpNQ32Refine { __device__ float operator()(float u) const { return normal_quantile_f32_refine(u); } };
struct OpNQ32Paper  { __device__ float operator()(float u) const { return normal_quantile_f32_paper(u); } };
struct OpNQ32Plain  { __device__ float operator()(float u) const { return normal_quantile_f32_plain(u); } };

/* Exponential -> normal in two parts: for every element, and for the rare
   ones beyond its range. */
struct OpE64Plain {
    static __device__ __forceinline__ double main(double x, bool* rare) { return exp_to_normal_f64_main(x, rare); }
    static __device__ __forceinline__ double rare(double x) { return exp_to_normal_f64_rare(x); }
};
struct OpE32Refine {
    static __device__ __forceinline__ float main(float x, bool* rare) { return exp_to_normal_f32_main(x, rare); }
    static __device__ __forceinline__ float rare(float x) { return exp_to_normal_f32_rare(x); }
};
struct OpE32Plain {
    static __device__ __forceinline__ float main(float x, bool* rare)
    {
        return (float)exp_to_normal_f64_main((double)x, rare);
    }
    static __device__ __forceinline__ float rare(float x) { return (float)exp_to_normal_f64_rare((double)x); }
};

/*
 * The hybrid quantiles (FP64 plain, FP32+refine) split each element into
 * the log-free central piece and the outer, exponential-coordinate path.
 * About 10% of uniform draws (and every element of a tail stratum) lie
 * outside the centre, so nearly every wave holds such a lane, and a wave
 * vote would cost every lane the outer path too.  The kernels instead give
 * every element the central piece, then gather the wave's outer elements
 * (hybrid_eval): each lane keeps K elements; the wave counts its outer elements (ballots),
 * writes their u to a per-wave LDS list at prefix-sum positions, evaluates
 * that list with one element per lane (one pass per 64) and reads each
 * result back.  The arithmetic on every element is that of the per-element
 * function (whole), so the results are bitwise identical to it.
 */
struct HybridNQ64 {
    typedef double T;
    /* central result into w; true if the element needs the outer path */
    static __device__ __forceinline__ bool split(double u, double& w)
    {
        double q = u - 0.5;
        w = central_quantile(q);
        return !is_central(q);
    }
    static __device__ __forceinline__ double outer(double u) { return outer_quantile_f64(u); }
    static __device__ __forceinline__ double whole(double u) { return normal_quantile_f64<false>(u); }
};

struct HybridNQ32 {
    typedef float T;
    static __device__ __forceinline__ bool split(float u, float& w)
    {
        double q = (double)u - 0.5;
        w = central_quantile_f32(q);
        return !is_central(q);
    }
    static __device__ __forceinline__ float outer(float u) { return outer_quantile_f32(u); }
    static __device__ __forceinline__ float whole(float u) { return normal_quantile_f32_refine(u); }
};

template <typename T> struct OpCopy { __device__ T operator()(T x) const { return x; } };

template <class Op> struct HybridOf { typedef void type; };
template <> struct HybridOf<OpNQ64Plain> { typedef HybridNQ64 type; };
template <> struct HybridOf<OpNQ32Refine> { typedef HybridNQ32 type; };

/* The gather step: u[K] per lane in, w[K] out; buf is the wave's LDS list
   of 64 K elements (its address must be wave-uniform).  Every lane of the
   wave must call it together.  Each slot's ballot is taken once, where its
   comparison is made, and kept as a scalar mask: a lane's list position is
   the running count (scalar) plus the set bits of that mask below the lane
   (two mbcnt), and the list address one shift-add from those. */
template <typename T, int K, class H>
__device__ __forceinline__ void hybrid_eval(const T (&u)[K], T (&w)[K], T* buf, uint32_t lane)
{
    bool outer[K];
    uint64_t m[K];
    uint32_t cnt = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        outer[k] = H::split(u[k], w[k]);
        m[k] = __ballot(outer[k]);
        cnt += (uint32_t)__popcll(m[k]);
    }
    if (!cnt) return;
    T* slot[K];
    uint32_t base = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], 0u));
        slot[k] = (buf + base) + below;
        if (outer[k]) *slot[k] = u[k];
        base += (uint32_t)__popcll(m[k]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t r = 0; r < base; r += 64) {
        if (r + lane < base) buf[r + lane] = H::outer(buf[r + lane]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (outer[k]) w[k] = *slot[k];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

/* A walk's map from a per-element function. */
template <typename T, class Op>
struct ElementMap {
    template <int K>
    __device__ __forceinline__ void tile(const T (&x)[K], T (&y)[K]) const
    {
        Op op;
#pragma unroll
        for (int k = 0; k < K; ++k) y[k] = op(x[k]);
    }
    __device__ __forceinline__ T one(T x) const { return Op()(x); }
};

/* A walk's map from a function in two parts: all of a lane's elements first
   (K independent chains; a vote between them would end each before the next
   begins), then one wave vote for the rare ones. */
template <typename T, class Op>
struct VotedMap {
    template <int K>
    __device__ __forceinline__ void tile(const T (&x)[K], T (&y)[K]) const
    {
        bool rare[K];
        bool any = false;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            y[k] = Op::main(x[k], &rare[k]);
            any |= rare[k];
        }
        if (wave_any(any)) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (wave_any(rare[k])) {
                    const T r = Op::rare(x[k]);
                    y[k] = rare[k] ? r : y[k];
                }
        }
    }
    __device__ __forceinline__ T one(T x) const
    {
        const T a[1] = {x};
        T y[1];
        tile(a, y);
        return y[0];
    }
};

template <typename T, class Op> struct MapOf { typedef ElementMap<T, Op> type; };
template <typename T> struct MapOf<T, OpE64Plain> { typedef VotedMap<T, OpE64Plain> type; };
template <typename T> struct MapOf<T, OpE32Refine> { typedef VotedMap<T, OpE32Refine> type; };
template <typename T> struct MapOf<T, OpE32Plain> { typedef VotedMap<T, OpE32Plain> type; };

/* A walk's map from a gathered hybrid; buf: the wave's LDS list. */
template <typename T, class H>
struct HybridMap {
    T* buf;
    uint32_t lane;
    template <int K>
    __device__ __forceinline__ void tile(const T (&x)[K], T (&y)[K]) const
    {
        hybrid_eval<T, K, H>(x, y, buf, lane);
    }
    __device__ __forceinline__ T one(T x) const { return H::whole(x); }
};

}  // namespace qm
