/*
 * qm_hyp_device.hpp -- device evaluation of the exponential -> hyperbolic
 * tables (Section 8.1; layout in qm_hyp_table.h), shared by the map kernel
 * (qm_hyp.hip) and the batch kernel (qm_batch.hip).
 */
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qm_device.hpp"
#include "qm_hyp_table.h"
#include "qm_stream.hpp"

namespace qm {

/* Rows of DEG + 1 doubles in global memory.  In LDS every row starts on a
   16-byte boundary and is read in 16-byte pieces (ds_read_b128), so lanes
   on different cells either share a 16-byte bank group or none: never a
   half overlap; and a row takes an odd number of such groups, so that the
   rows start in every one of them.  FP64-output cells (degree 11): twelve
   doubles padded to fourteen, six reads.  Where the caches feed the map the
   LDS reads are its limit: 2^22 samples of (1, 0.5, 1) take 13.8 us on
   MI355X against 14.8 with rows of twelve, whose starts miss half the
   groups, 2^20 5.6 against 6.2; from 2^26 on both stream at the memory's
   rate.  FP32-output cells (degree 7) are stored mixed: the constant term as
   a double (dwords 0-1), the seven higher coefficients as floats, highest
   power first (dwords 2-8), padded to 12 dwords: two 16-byte reads and one
   4-byte read (36 bytes, against 64 for eight doubles).  lds is the row
   stride in doubles.  The dynamic LDS the rows live in is declared 16-byte
   aligned. */
template <int DEG> struct HypRow {
    static constexpr int n = DEG + 1;
    static constexpr int lds = DEG == HYP_DEGREE_F32 ? 6 : DEG + 3;
    static_assert(lds % 4 == 2, "rows must take an odd number of 16-byte groups");
};
static_assert(HYP_SUB == 8, "the cell index takes the top 3 mantissa bits of t");

/* The far path's parameters of one side. */
struct HypSideFar {
    double v_top, c0, c1, c2, clog;
    const double* gcoef;          /* the side's rows in global memory */
    int ncell;
};

struct HypParams {
    double v0, inv_v0, mu;        /* v0 is shared by both sides */
    HypSideFar r, l;              /* v >= 0, v < 0 */
    int nlds;                     /* cells per side in LDS, right side's first */
    int jlo;                      /* first cell the LDS path takes: 0, or HYP_SUB when the sides
                                     hold the origin series in their first octave; both sides'
                                     series then follow the cells in LDS, as the doubles of row 0 */
};


/* Cell of t = 1 + a/v0 >= 1: the biased exponent and the top three mantissa
   bits of t give j = 8 k + i for t in [2^k (1 + i/8), 2^k (1 + (i+1)/8));
   the cell's centre in t, 2^k (1 + (i + 1/2)/8), is t with the lower
   mantissa bits replaced by 1000...  NaN and inf give j >= 8192. */
__device__ __forceinline__ int hyp_cell(double t, double* tc)
{
    const uint32_t hi = (uint32_t)__double2hiint(t);
    *tc = __hiloint2double((int)((hi & ~((1u << 17) - 1)) | (1u << 16)), 0);
    return (int)(hi >> 17) - (1023 << 3);
}

template <int DEG>
__device__ __forceinline__ double hyp_poly(const double* __restrict__ c, double d)
{
    double R = c[0];
#pragma unroll
    for (int k = 1; k <= DEG; ++k) R = __builtin_fma(R, d, c[k]);
    return R;
}

/*
 * R of LDS row `row` at d.  FP64-output cells: Horner in FP64.  FP32-output
 * cells: R = c0 + d S(d), S the seven higher terms by Horner in FP32 from
 * float coefficients, c0 and the last step in FP64.  Across every cell the
 * builder produces, |R - c0| stays a small part of |R| (below 6% for the
 * parameters tested), so the FP32 part adds a relative error of about
 * 0.06 x 2^-22 to R, far below the half-ulp of the FP32 result.
 */
template <int DEG>
__device__ __forceinline__ double hyp_cell(const double* __restrict__ lds, int row, double d)
{
    if constexpr (DEG == HYP_DEGREE_F32) {
        typedef float f4v __attribute__((ext_vector_type(4)));
        typedef double d2v __attribute__((ext_vector_type(2)));
        const double* r = lds + __umul24((uint32_t)row, (uint32_t)HypRow<DEG>::lds);
        const d2v a = *reinterpret_cast<const d2v*>(r);            /* c0, then the top two floats */
        const f4v b = *reinterpret_cast<const f4v*>(r + 2);
        const float last = reinterpret_cast<const float*>(r + 4)[0];
        const double c0 = a.x;
        const float f0 = __int_as_float(__double2loint(a.y)), f1 = __int_as_float(__double2hiint(a.y));
        const float df = (float)d;
        float S = __builtin_fmaf(f0, df, f1);
        S = __builtin_fmaf(S, df, b.x);
        S = __builtin_fmaf(S, df, b.y);
        S = __builtin_fmaf(S, df, b.z);
        S = __builtin_fmaf(S, df, b.w);
        S = __builtin_fmaf(S, df, last);
        return __builtin_fma(d, (double)S, c0);
    } else {
        typedef double d2v __attribute__((ext_vector_type(2)));
        const double* r = lds + __umul24((uint32_t)row, (uint32_t)HypRow<DEG>::lds);
        double c[DEG + 1];
#pragma unroll
        for (int k = 0; k < (DEG + 1) / 2; ++k) {
            const d2v x = *reinterpret_cast<const d2v*>(r + 2 * k);
            c[2 * k] = x.x;
            c[2 * k + 1] = x.y;
        }
        return hyp_poly<DEG>(c, d);
    }
}

/* |Q(v)| from the LDS cells; *far for lanes beyond them (and NaN). */
template <int DEG>
__device__ __forceinline__ double hyp_near(double v, const double* __restrict__ lds, const HypParams& P, bool* far)
{
    const double a = __builtin_fabs(v);
    const double t = __builtin_fma(a, P.inv_v0, 1.0);
    double tc;
    int j = hyp_cell(t, &tc);                    /* >= 0: t >= 1 */
    const bool out = !((unsigned)(j - P.jlo) < (unsigned)(P.nlds - P.jlo));
    *far = out;
    j = out ? P.nlds - 1 : j;                     /* far and NaN lanes stay in bounds */
    const int row = j + (v < 0.0 ? P.nlds : 0);
    const double d = __builtin_fma(-P.v0, tc - 1.0, a);   /* a - centre; tc - 1 is exact */
    return a * hyp_cell<DEG>(lds, row, d);
}

/*
 * a^rho for 0 < a <= 1, rho > 0, within 3e-16 relative.  log a = hi + lo to
 * about 1e-18 absolute: a = m 2^e with m in [sqrt(1/2), sqrt(2)), log m =
 * 2 atanh f as in neg_log_unit, with the remainders of f, of m + 1 and of the
 * sum with e log 2 carried; an absolute error of rho log a is a relative one
 * of the power, and |rho log a| reaches hundreds.  Then e^(hi + lo) = 2^k e^r,
 * e^r by its Taylor polynomial of degree 13 (remainder 4e-18).  rcp: a
 * reciprocal good to 5e-8.  a = 0 gives some finite value.  A logarithm and
 * an exponential with no remainders were up to 1.2e-14 off in the power at
 * rho = 7.5 for a not far below v0, 5.8e-14 at a^rho = 1e-300.  Variance-gamma
 * (4.25, 1, 0.3), 2^24 samples on MI355X: FP64 50.7 us without the remainders,
 * 51.2 with them, 56.5 with the library pow; FP32 32.7, 33.8 and 43.
 */
template <class Rcp>
__host__ __device__ __forceinline__ double pow_small(double a, double rho, Rcp rcp)
{
    const double SQRT_HALF = 0.70710678118654752440, LOG2E = 1.4426950408889634074;
    const double LN2_HI = 6.93147180369123816490e-01, LN2_LO = 1.90821492927058770002e-10;     /* e LN2_HI is exact */
    const double LN2_D = 0.69314718055994528623, LN2_E = 2.3190468138462996154e-17;            /* ln 2 as two doubles */
    int e;
    double m = __builtin_frexp(a, &e);
    const int up = m < SQRT_HALF;
    m = __builtin_ldexp(m, up);
    const double de = (double)(e - up);
    const double n1 = m + 1.0, n2 = m - (n1 - 1.0);                 /* m + 1 = n1 + n2 */
    double y = rcp(n1);
    y = __builtin_fma(__builtin_fma(-n1, y, 1.0), y, y);
    const double f0 = (m - 1.0) * y;
    const double df = __builtin_fma(-f0, n2, __builtin_fma(-f0, n1, m - 1.0)) * y;
    const double f = f0 + df, f_lo = df - (f - f0);                 /* (m - 1) / (m + 1) = f + f_lo */
    double p = QM_LOG_R[0];
    const double s = f * f, t = f + f, eh = de * LN2_HI;
#pragma unroll
    for (int i = 1; i < 7; ++i) p = __builtin_fma(p, s, QM_LOG_R[i]);
    const double hi = eh + t;                                       /* |eh| >= |t|, or eh = 0 */
    const double lo = (t - (hi - eh)) + __builtin_fma(de, LN2_LO, __builtin_fma(f * s, p, f_lo + f_lo));
    const double x = rho * hi, x_lo = __builtin_fma(rho, lo, __builtin_fma(rho, hi, -x));
    const double k = __builtin_rint(x * LOG2E);
    const double r = __builtin_fma(-k, LN2_D, x) + __builtin_fma(-k, LN2_E, x_lo);
    double fact = 6227020800.0;                                     /* 13!, folded with the loop */
    double w = 1.0 / fact;
#pragma unroll
    for (int i = 13; i >= 1; --i) {
        fact /= i;
        w = __builtin_fma(w, r, 1.0 / fact);
    }
    return __builtin_ldexp(w, (int)k);
}

/* |Q(a)| in the first octave of a side with the origin series (row 0 of its
   cells, layout in qm_hyp_table.h; here in LDS): a R, R = P0(a) + w (P1(a) +
   w (P2(a) + w P3(a))), w = a^rho; FP32-output cells have no P3.  Out of line:
   a kernel's loop would hold its constants otherwise. */
typedef const __attribute__((address_space(3))) double* LdsRow;
template <int DEG>
static __device__ __noinline__ double hyp_origin(LdsRow row, double a)
{
    /* the families in row order, from the highest power of w down, and
       their degrees in v */
    constexpr int NFAM = DEG == HYP_DEGREE ? 4 : 3;
    constexpr int DG64[4] = {0, 1, 2, 4}, DG32[4] = {0, 1, 3, 0};
    const double w = pow_small(a, row[0], [](double x) { return __builtin_amdgcn_rcp(x); });
    double R = 0;
    int k = 1;
#pragma unroll
    for (int n = 0; n < NFAM; ++n) {
        const int dg = DEG == HYP_DEGREE ? DG64[n] : DG32[n];
        double p = 0;
#pragma unroll
        for (int m = 0; m <= dg; ++m, ++k) p = __builtin_fma(p, a, row[k]);
        R = __builtin_fma(R, w, p);
    }
    return a * R;
}

/* |Q(v)| beyond the LDS cells: the side's global-memory cells up to v_top,
   then the large-v form; inf -> inf, NaN -> NaN.  The side's parameters come as plain values
   selected per lane (a reference to a lane-dependent side, or a struct
   passed by value, would put them in scratch memory). */
template <int DEG>
static __device__ __noinline__ double hyp_far(double a, double v0, double inv_v0, double v_top, double c0, double c1,
                                              double c2, double clog, const double* gcoef, int ncell)
{
    if (!(a < v_top)) {
        if (!(a < __builtin_inf())) return a;
        if (clog == 0.0) return a + (c0 + (c1 + c2 / a) / a);
        /* a tail with a power of x: Q = a + c0 + clog log Q + (c1 + c2/Q)/Q,
           three fixed-point steps (each gains a factor clog/Q) */
        double q = a + c0 - clog * neg_log_unit(a);
        for (int i = 0; i < 3; ++i) q = a + c0 - clog * neg_log_unit(q) + (c1 + c2 / q) / q;
        return q;
    }
    double tc;
    int j = hyp_cell(__builtin_fma(a, inv_v0, 1.0), &tc);
    j = (unsigned)j < (unsigned)ncell ? j : ncell - 1;
    return a * hyp_poly<DEG>(gcoef + j * HypRow<DEG>::n, __builtin_fma(-v0, tc - 1.0, a));
}

template <int DEG>
__device__ __forceinline__ double hyp_far_of(double v, const HypParams& P)
{
    const bool neg = v < 0.0;
    return hyp_far<DEG>(__builtin_fabs(v), P.v0, P.inv_v0, neg ? P.l.v_top : P.r.v_top, neg ? P.l.c0 : P.r.c0,
                   neg ? P.l.c1 : P.r.c1, neg ? P.l.c2 : P.r.c2, neg ? P.l.clog : P.r.clog,
                   neg ? P.l.gcoef : P.r.gcoef, neg ? P.l.ncell : P.r.ncell);
}

/* Both sides' LDS rows: right side rows 0..nlds-1, left side after (for
   the FP32-output cells in the mixed layout of HypRow).  16-byte loads (the
   rows in device memory are 8-byte aligned), four of a thread's in flight
   together: an FP64 row's twelve doubles are six pieces; an FP32-output row
   of eight doubles goes to one thread, which writes its three 16-byte
   groups. */
template <int DEG>
__device__ __forceinline__ void stage_hyp(double* lds, const HypParams& P)
{
    typedef double d2any __attribute__((ext_vector_type(2), aligned(8)));
    typedef double d2v __attribute__((ext_vector_type(2)));
    constexpr int PIECES = HypRow<DEG>::n / 2;
    const int step = blockDim.x;
    if (P.jlo && threadIdx.x < 2 * HypRow<DEG>::n) {
        const int left = threadIdx.x >= HypRow<DEG>::n, k = threadIdx.x - left * HypRow<DEG>::n;
        lds[2 * P.nlds * HypRow<DEG>::lds + threadIdx.x] = (left ? P.l.gcoef : P.r.gcoef)[k];
    }
    if constexpr (DEG == HYP_DEGREE_F32) {
        typedef float f4v __attribute__((ext_vector_type(4)));
        for (int r = threadIdx.x; r < 2 * P.nlds; r += step) {
            const double* src = r < P.nlds ? P.r.gcoef + r * HypRow<DEG>::n : P.l.gcoef + (r - P.nlds) * HypRow<DEG>::n;
            d2any c[PIECES];
#pragma unroll
            for (int k = 0; k < PIECES; ++k) c[k] = reinterpret_cast<const d2any*>(src)[k];
            double* row = lds + r * HypRow<DEG>::lds;
            d2v head;
            head.x = c[3].y;
            head.y = __hiloint2double(__float_as_int((float)c[0].y), __float_as_int((float)c[0].x));
            *reinterpret_cast<d2v*>(row) = head;
            *reinterpret_cast<f4v*>(row + 2) = f4v{(float)c[1].x, (float)c[1].y, (float)c[2].x, (float)c[2].y};
            reinterpret_cast<float*>(row + 4)[0] = (float)c[3].x;
        }
    } else {
        const int n = P.nlds * PIECES;
        for (int i = threadIdx.x; i < 2 * n; i += 4 * step) {
            d2any v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = min(i + k * step, 2 * n - 1);
                v[k] = reinterpret_cast<const d2any*>(e < n ? P.r.gcoef : P.l.gcoef)[e < n ? e : e - n];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = i + k * step;
                if (e < 2 * n)
                    reinterpret_cast<d2v*>(lds)[e / PIECES * (HypRow<DEG>::lds / 2) + e % PIECES] = v[k];
            }
        }
    }
}

/* One pass over a lane's flagged elements: f of the first of them (bit `bit`
   of the K), and its result in its place. */
template <int K, class F>
__device__ __forceinline__ void one_per_lane(const double (&v)[K], double (&q)[K], uint32_t& left, F f)
{
    const uint32_t bit = left & -left;
    double x = 0.0;
#pragma unroll
    for (int e = 0; e < K; ++e) x = (bit >> e) & 1u ? v[e] : x;
    const double r = f(x);
#pragma unroll
    for (int e = 0; e < K; ++e) q[e] = (bit >> e) & 1u ? r : q[e];
    left ^= bit;
}

/*
 * |Q(v)| of the K elements a lane holds: every element's cell polynomial
 * first (K independent chains), then, if any lane of the wave has elements
 * beyond the LDS cells, passes that take one such element of each lane at a
 * time, whichever of the K it is.  Such elements are rare and scattered: on a
 * target with the origin series about 0.2% of the base samples are, so that a
 * wave's tile of 512 holds one on average in one or two lanes, and one
 * pass serves it.  A vote for each of the K slots entered the far code once
 * per slot that held any, with the series' row from device memory and a
 * library pow each (2^24 FP64 samples of variance-gamma (4.25, 1, 0.3): 67.2
 * us on MI355X; 52.5 with the passes and a short power, 49.7 with the rows
 * in LDS).
 */
template <int DEG, int K>
__device__ __forceinline__ void hyp_abs_q(const double (&v)[K], double (&q)[K], const double* __restrict__ lds,
                                          const HypParams& P)
{
    bool far[K];
    bool anyfar = false;
#pragma unroll
    for (int e = 0; e < K; ++e) {
        q[e] = hyp_near<DEG>(v[e], lds, P, &far[e]);
        anyfar |= far[e];
    }
    if (wave_any(anyfar)) {
        uint32_t left = 0;
#pragma unroll
        for (int e = 0; e < K; ++e) left |= far[e] ? 1u << e : 0u;
        if (P.jlo) {
            uint32_t first = 0;
#pragma unroll
            for (int e = 0; e < K; ++e) first |= far[e] && __builtin_fabs(v[e]) < P.v0 ? 1u << e : 0u;
            left ^= first;
            const LdsRow series = (LdsRow)(lds + 2 * P.nlds * HypRow<DEG>::lds);
            while (wave_any(first != 0))
                one_per_lane(v, q, first, [&](double x) {
                    return hyp_origin<DEG>(series + (x < 0.0 ? HypRow<DEG>::n : 0), __builtin_fabs(x));
                });
        }
        while (wave_any(left != 0)) one_per_lane(v, q, left, [&](double x) { return hyp_far_of<DEG>(x, P); });
    }
}

/* A walk's map of the hyperbolic and variance-gamma targets:
   x = mu + sign(v) |Q(v)|, in FP64; FP32 outputs round it once. */
template <typename T, int DEG>
struct HypMap {
    const double* lds;
    const HypParams& P;
    template <int K>
    __device__ __forceinline__ void tile(const T (&x)[K], T (&y)[K]) const
    {
        constexpr int C = K > 8 ? 8 : K;    /* eight chains at a time: sixteen cost half the occupancy */
#pragma unroll
        for (int c = 0; c < K; c += C) {
            double v[C], q[C];
#pragma unroll
            for (int k = 0; k < C; ++k) v[k] = (double)x[c + k];
            hyp_abs_q<DEG, C>(v, q, lds, P);
#pragma unroll
            for (int k = 0; k < C; ++k) y[c + k] = (T)(P.mu + __builtin_copysign(q[k], v[k]));
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

/* Kernel parameters of a table's cell set for FP64 (f32 = false) or FP32
   outputs (qm_hyp.hip): false if the header is not a valid table of ncoef
   doubles.  *lds_bytes gets the LDS the staged cells take. */
bool make_hyp_params(const HypTableHeader& h, bool f32, const HypTableHeader* d_table, uint64_t ncoef, double mu,
                     HypParams* P, size_t* lds_bytes);

}  // namespace qm
