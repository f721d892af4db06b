/*
 * qm_student_device.hpp -- per-element evaluation of the normal -> Student t
 * map from a table staged in LDS (shared by the single-request and the
 * batch kernels).
 */
#pragma once
#include <hip/hip_runtime.h>

#include "qm_device.hpp"
#include "qm_stream.hpp"

namespace qm {

/* Uniform per-launch parameters: the tail constants of the table header and
   the layout of the cell approximation in use. */
struct StudentParams {
    double h, inv_h, centre_offset, y_lds, y_max, log_K, tail_a, sqrt_nu, nu;
    const double* gcoef;  /* all ncell rows in global memory (the rare path reads them) */
    int ncell;        /* rows covering y <= y_max */
    int nlds;         /* rows staged in LDS, covering y <= y_lds */
    int identity;
    int row_shift;    /* log2 of the coefficients per row in memory (degree + 1) */
    int lds_stride;   /* doubles between cell rows in LDS: even, >= the row */
};

/* 16 bytes at the alignment of a double (gfx950 takes a dwordx4 load at any
   dword): table rows in device memory follow a header of 8-byte multiples. */
typedef double d2any __attribute__((ext_vector_type(2), aligned(8)));

inline size_t student_lds_bytes(const StudentParams& P) { return (size_t)P.nlds * P.lds_stride * sizeof(double); }

/* Copy the first nlds cell rows (2^row_shift doubles each) into LDS rows of
   P.lds_stride doubles, in 16-byte pieces, four in flight per thread before
   the first is waited for: a workgroup's staging is then one or two trips to
   the L2 instead of a chain of six to twelve 8-byte ones. */
__device__ __forceinline__ void stage_table(double* lds, const double* __restrict__ coef, const StudentParams& P)
{
    const int shift = P.row_shift - 1;              /* pieces per row */
    const int n = P.nlds << shift;
    const int mask = (1 << shift) - 1;
    const d2any* src = reinterpret_cast<const d2any*>(coef);
    const int step = blockDim.x;
    for (int i = threadIdx.x; i < n; i += 4 * step) {
        d2any v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = src[min(i + k * step, n - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int e = i + k * step;
            if (e < n) *reinterpret_cast<d2*>(lds + (e >> shift) * P.lds_stride + 2 * (e & mask)) = v[k];
        }
    }
}

/* R(y) of cell j by Horner in d = y - y_c (rows of DEG + 1 doubles). */
template <int DEG>
__device__ __forceinline__ double cell_poly(const double* __restrict__ c, double d)
{
    double R = c[0];
#pragma unroll
    for (int k = 1; k <= DEG; ++k) R = __builtin_fma(R, d, c[k]);
    return R;
}

/* The same from a row in LDS, read in 16-byte pieces (ds_read_b128): the
   rows start on 16-byte boundaries (even stride, 16-byte aligned LDS), so
   lanes on different cells either share a 16-byte bank group or none. */
template <int DEG>
__device__ __forceinline__ double cell_poly_lds(const double* __restrict__ row, double d)
{
    static_assert((DEG + 1) % 2 == 0, "rows of an even number of doubles");
    typedef double d2v __attribute__((ext_vector_type(2)));
    double c[DEG + 1];
#pragma unroll
    for (int k = 0; k < (DEG + 1) / 2; ++k) {
        const d2v x = *reinterpret_cast<const d2v*>(row + 2 * k);
        c[2 * k] = x.x;
        c[2 * k + 1] = x.y;
    }
    return cell_poly<DEG>(c, d);
}

/* Cell index and offset for s = |z|: j from y = s^2 by one multiply,
   clamped to jmax (NaN and inf clamp too), and d = s^2 - y_c with a single
   rounding (|d| <= h/2), so the full input precision reaches the
   polynomial, which matters because log R grows like y/(2 nu). */
__device__ __forceinline__ int cell_of(double s, double yh, int jmax, double h, double inv_h, double centre_offset,
                                       double* d)
{
    int j = (int)__builtin_fmin(yh * inv_h, (double)jmax);
    double yc = __builtin_fma((double)j, h, centre_offset);   /* exact: h is a power of 2 */
    *d = __builtin_fma(s, s, -yc);
    return j;
}

/* Beyond the LDS cells (y > y_lds, |z| above about 10).  Up to y_max the
   remaining cells, from global memory.  Beyond: w = K q(s),
   q(s) = erfcx(s/sqrt2) e^{-s^2/2} / 2, t = sqrt(nu) w^{-1/nu} (1 + a w^{2/nu})
   (Sections 3.3, 3.5), which the table builder has checked to be as accurate
   as the cells there.  log w is carried as a double-double (s^2/2 exactly,
   the division by nu with its remainder), because an absolute error e in it
   is a relative error e/nu in t and |log w| reaches several hundred.  The
   parameters come one by one: a reference to the block of them put a copy of
   it in every lane's scratch memory at the head of the kernel, 128 bytes per
   element of a short launch. */
template <int DEG>
static __device__ __noinline__ double student_far(double s, double h, double inv_h, double centre_offset, double y_max,
                                                  const double* gcoef, int ncell, double log_K, double nu,
                                                  double sqrt_nu, double tail_a)
{
#pragma clang fp contract(off)
    const double INV_SQRT2 = 0.70710678118654752440, LN2 = 0.69314718055994530942;
    if (!(s < __builtin_inf())) return s;              /* z = +-inf -> +-inf; NaN -> NaN */
    double yh = s * s;
    /* s^2 overflows (s above 1.3e154): log t is about s^2/(2 nu) > 700 for
       every nu below 1e300, so t overflows too */
    if (!(yh < __builtin_inf())) return yh;
    if (yh <= y_max) {
        double d;
        int j = cell_of(s, yh, ncell - 1, h, inv_h, centre_offset, &d);
        return s * cell_poly<DEG>(gcoef + j * (DEG + 1), d);
    }
    double hs = -0.5 * s;                              /* exact */
    double e_hi = hs * s;
    double e_lo = __builtin_fma(hs, s, -e_hi);         /* -s^2/2 = e_hi + e_lo exactly */
    double r = log_K + (::log(::erfcx(s * INV_SQRT2)) - LN2);
    double a_hi = e_hi + r;                            /* two-sum */
    double bb = a_hi - e_hi;
    double a_lo = (e_hi - (a_hi - bb)) + (r - bb) + e_lo;
    double q_hi = a_hi / nu;                           /* log w / nu = q_hi + q_lo */
    double q_lo = (__builtin_fma(-q_hi, nu, a_hi) + a_lo) / nu;
    double t = sqrt_nu * ::exp(-q_hi) * (1.0 - q_lo);
    return t * (1.0 + tail_a * ::exp(2.0 * q_hi));
}

/* t(z) in FP64, from the LDS table with cells of degree DEG, of the K
   elements a lane holds: K independent chains, then one wave vote for the
   elements beyond the LDS cells (also NaN, which propagates either way), of
   which a pass takes one of each lane. */
template <int DEG, int K>
__device__ __forceinline__ void student_eval(const double (&z)[K], double (&t)[K], const double* __restrict__ tab,
                                             const StudentParams& P)
{
    bool far[K];
    bool anyfar = false;
#pragma unroll
    for (int e = 0; e < K; ++e) {
        const double s = __builtin_fabs(z[e]);
        const double yh = s * s;            /* only selects the cell */
        double d;
        const int j = cell_of(s, yh, P.nlds - 1, P.h, P.inv_h, P.centre_offset, &d);
        t[e] = z[e] * cell_poly_lds<DEG>(tab + __umul24((uint32_t)j, (uint32_t)P.lds_stride), d);
        far[e] = !(yh <= P.y_lds);
        anyfar |= far[e];
    }
    if (wave_any(anyfar)) {
        uint32_t left = 0;
#pragma unroll
        for (int e = 0; e < K; ++e) left |= far[e] ? 1u << e : 0u;
        do {
            const uint32_t bit = left & -left;
            double x = 1.0;
#pragma unroll
            for (int e = 0; e < K; ++e) x = (bit >> e) & 1u ? z[e] : x;
            double f = student_far<DEG>(__builtin_fabs(x), P.h, P.inv_h, P.centre_offset, P.y_max, P.gcoef, P.ncell,
                                        P.log_K, P.nu, P.sqrt_nu, P.tail_a);
            f = __builtin_copysign(f, x);
#pragma unroll
            for (int e = 0; e < K; ++e) t[e] = (bit >> e) & 1u ? f : t[e];
            left ^= bit;
        } while (wave_any(left != 0));
    }
}

/* A walk's map of Student t.  FP32 in/out: the FP64 evaluation of the
   table's FP32 cells (R to 1e-10) rounded once; the input is exact in FP64,
   so the cell offset carries the input's full precision. */
template <typename T, int DEG>
struct StudentMap {
    const double* tab;
    const StudentParams& P;
    template <int K>
    __device__ __forceinline__ void tile(const T (&x)[K], T (&y)[K]) const
    {
        constexpr int C = K > 8 ? 8 : K;    /* eight chains at a time: sixteen cost half the occupancy */
#pragma unroll
        for (int c = 0; c < K; c += C) {
            double z[C], t[C];
#pragma unroll
            for (int k = 0; k < C; ++k) z[k] = (double)x[c + k];
            student_eval<DEG, C>(z, t, tab, P);
#pragma unroll
            for (int k = 0; k < C; ++k) y[c + k] = (T)t[k];
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

}  // namespace qm
