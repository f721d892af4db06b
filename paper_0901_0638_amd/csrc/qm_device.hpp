/*
 * qm_device.hpp -- per-element device math for gfx950 (wave64).
 *
 * Everything here is branch-free per lane.  The only control flow is
 * wave-uniform: a rare piece (the deep tail beyond the paper's v = 42) is
 * entered when any lane of the wave needs it, decided by a wave vote, so no
 * lane ever diverges from its neighbours (the paper's warp-vote idea,
 * Section 7.3, applied to the tail instead of the centre).
 */
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qm_coeffs.h"
#include "qm_paper_coeffs.h"

namespace qm {

/* Horner chain p <- p x + c, highest power first (Section 4.5.1: FMA-friendly
   iterated linear maps, no quadratic factorisation). */
template <int N>
__device__ __forceinline__ double horner(double x, const double (&c)[N])
{
    double acc = c[0];
#pragma unroll
    for (int i = 1; i < N; ++i) acc = __builtin_fma(acc, x, c[i]);
    return acc;
}

/*
 * The coefficients of the outer quantile pieces, in constant memory.  Their
 * chains are too long for the scalar registers beside a kernel's loop; held
 * in vector registers instead, each is first copied into the accumulator of a
 * two-operand v_fmac_f64, one v_mov_b64 for every step (21 of the 66
 * instructions of the FP32 piece, of the 111 of the FP64 one).  Loaded where
 * they are used (scalar loads, from an address the compiler cannot see
 * through, or it would hoist them out of the loop again) and given to
 * v_fma_f64 as its scalar operand, which the compiler would not do by itself,
 * every step is one instruction, and the kernels need 52 to 69 vector
 * registers where they needed 85 to 107.  MI355X, per pass: 2^26
 * mixture quantiles 102.2 -> 98.0 us in FP32, 2^28 in FP64 767 -> 751, 2^26
 * fused FP32 quantiles 94.4 -> 91.7.
 */
struct OuterCoeffs {
    double p13[14], q13[14], tail_p[8], tail_q[8], log_r[7];   /* FP64 */
    double log32[11], p32[8], q32[8];                          /* FP32 */
};
template <int N>
constexpr void copy_coeffs(double (&to)[N], const double (&from)[N])
{
    for (int i = 0; i < N; ++i) to[i] = from[i];
}
constexpr OuterCoeffs outer_coeffs()
{
    OuterCoeffs c{};
    copy_coeffs(c.p13, QM_PAPER_P13);
    copy_coeffs(c.q13, QM_PAPER_Q13);
    copy_coeffs(c.tail_p, QM_TAIL_P);
    copy_coeffs(c.tail_q, QM_TAIL_Q);
    copy_coeffs(c.log_r, QM_LOG_R);
    copy_coeffs(c.log32, QM_D32_LOG);
    copy_coeffs(c.p32, QM_D32_OP);
    copy_coeffs(c.q32, QM_D32_OQ);
    return c;
}
static __constant__ const OuterCoeffs QM_OUTER = outer_coeffs();

typedef const __attribute__((address_space(4))) OuterCoeffs* OuterPtr;
__device__ __forceinline__ OuterPtr outer_ptr()
{
    OuterPtr c = (OuterPtr)&QM_OUTER;
    asm volatile("" : "+s"(c));
    return c;
}

template <int N>
__device__ __forceinline__ double horner(double x, const __attribute__((address_space(4))) double (&c)[N])
{
    double acc = c[0];
#pragma unroll
    for (int i = 1; i < N; ++i) asm("v_fma_f64 %0, %1, %2, %3" : "=v"(acc) : "v"(acc), "v"(x), "s"(c[i]));
    return acc;
}

template <int N>
__device__ __forceinline__ float hornerf(float x, const float (&c)[N])
{
    float acc = c[0];
#pragma unroll
    for (int i = 1; i < N; ++i) acc = __builtin_fmaf(acc, x, c[i]);
    return acc;
}

/* a / b for finite positive b of moderate size.  The hardware reciprocal is
   good to ~5e-8, so one Newton step on it (error ~2e-15) and one residual
   correction of the quotient give a result within an ulp. */
__device__ __forceinline__ double div_pos(double a, double b)
{
    double y = __builtin_amdgcn_rcp(b);
    double e = __builtin_fma(-b, y, 1.0);
    y = __builtin_fma(e, y, y);
    double q = a * y;
    double r = __builtin_fma(-b, q, a);
    return __builtin_fma(r, y, q);
}

/* sqrt(v) for positive normal v, within an ulp: hardware reciprocal square
   root (~5e-8), one coupled Newton step on (sqrt v, 1/(2 sqrt v)), one
   residual correction.  Other inputs give unspecified values. */
__device__ __forceinline__ double sqrt_pos(double v)
{
    double r = __builtin_amdgcn_rsq(v);
    double s = v * r, h = 0.5 * r;
    double e = __builtin_fma(-s, h, 0.5);
    s = __builtin_fma(s, e, s);
    h = __builtin_fma(h, e, h);
    double d = __builtin_fma(-s, s, v);
    return __builtin_fma(d, h, s);
}

/* c ? a : b with the lane mask in a scalar register pair.  The compiler keeps
   a select's mask in VCC, where a second v_cndmask_b32 straight after the
   first takes 23 cycles a wave on gfx950; a 64-bit select is two of them (25
   cycles with its comparison, 11 through a scalar pair).  In the FP64 paths a
   minimum, a ldexp by the comparison's 0 or 1, or an added special takes the
   place of a select where one can: 2^24 fused samples, hyperbolic FP64 63.6 ->
   61.1 us and FP32 49.2 -> 46.8, Student t FP64 57.8 -> 56.4. */
__device__ __forceinline__ double select_f64(bool c, double a, double b)
{
    uint64_t m = __builtin_amdgcn_ballot_w64(c);
    asm("" : "+s"(m));
    return __builtin_amdgcn_inverse_ballot_w64(m) ? a : b;
}

/* -log(x) for x in (0, 1], relative error about an ulp.  x = m 2^e with m in
   [sqrt(1/2), sqrt(2)); log m = 2 atanh f = 2f + f s R(s), f = (m-1)/(m+1)
   (exact numerator), s = f^2, R a fitted degree-6 polynomial; log 2 is split
   so that e log2_hi is exact.  Denormal x is handled by frexp.  x = 0,
   negative or NaN x give unspecified values: callers select their results. */
template <class R>
__device__ __forceinline__ double neg_log_unit(double x, const R& coeffs)
{
    const double SQRT_HALF = 0.70710678118654752440;
    const double LN2_HI = 6.93147180369123816490e-01, LN2_LO = 1.90821492927058770002e-10;
    double m = __builtin_amdgcn_frexp_mant(x);
    int e = __builtin_amdgcn_frexp_exp(x);
    const int lo = m < SQRT_HALF;            /* a scaling by 2^lo: cheaper than 64-bit selects */
    m = __builtin_amdgcn_ldexp(m, lo);
    e -= lo;
    double f = div_pos(m - 1.0, m + 1.0);
    double s = f * f;
    double lm = __builtin_fma(f * s, horner(s, coeffs), f + f);
    double de = (double)e;
    return -__builtin_fma(de, LN2_HI, __builtin_fma(de, LN2_LO, lm));
}

__device__ __forceinline__ double neg_log_unit(double x) { return neg_log_unit(x, QM_LOG_R); }

/* any lane of the wave */
__device__ __forceinline__ bool wave_any(bool p) { return __any((int)p) != 0; }

/* ------------------------------------------------------------------------ */
/* Exponential-coordinate normal quantile Q(v) = Phi^{-1}(1 - e^{-v}/2),     */
/* v >= 0 (Section 6 formal solution; Section 7.2 branchless rational).      */
/* ------------------------------------------------------------------------ */

/* v > 750 (only reachable through exp -> normal with |x| > 750): from the
   Mills-ratio expansion of the normal tail, log q(z) = -z^2/2 - log(z sqrt(2 pi))
   + log S(z), S = 1 - z^-2 + 3 z^-4 - 15 z^-6 + 105 z^-8, solve
   z^2 = 2 (v + log 2 - log(z sqrt(2 pi)) + log S(z)) by fixed-point
   iteration; the map contracts by ~1/z^2 < 1/1500 per step. */
__device__ __noinline__ double expcoord_far(double v)
{
    const double LN2 = 0.69314718055994530942, LN_SQRT2PI = 0.91893853320467274178;
    double z = __builtin_sqrt(2.0) * __builtin_sqrt(v);
    for (int k = 0; k < 5; ++k) {
        double iz2 = 1.0 / (z * z);
        double S = __builtin_fma(__builtin_fma(__builtin_fma(105.0 * iz2 - 15.0, iz2, 3.0), iz2, -1.0), iz2, 1.0);
        double L = ::log(z) + LN_SQRT2PI - ::log(S);
        z = __builtin_sqrt(2.0) * __builtin_sqrt(v + (LN2 - L));
    }
    return z;
}

/* Plain FP64 Q(v) for v in [0, 750]: the paper's (13,13) rational on v <= 42
   and the fitted Q(v) = s P7(s)/Q7(s), s = sqrt v, beyond.  Both pieces end in
   a single division. */
__device__ __forceinline__ double expcoord_q_plain(double v, OuterPtr c)
{
    double num = v * horner(v, c->p13);
    double den = horner(v, c->q13);
    bool tail = v > QM_TAIL_VMIN;
    if (wave_any(tail)) {
        double s = sqrt_pos(v);
        double nt = s * horner(s, c->tail_p);
        double dt = horner(s, c->tail_q);
        num = select_f64(tail, nt, num);
        den = select_f64(tail, dt, den);
    }
    return div_pos(num, den);
}

/* Paper mode: the (13,13) rational verbatim, whatever v (Appendix B). */
__device__ __forceinline__ double expcoord_q_paper(double v)
{
    return div_pos(v * horner(v, QM_PAPER_P13), horner(v, QM_PAPER_Q13));
}

/* ------------------------------------------------------------------------ */
/* FP64 normal quantile w(u) = Phi^{-1}(u).                                  */
/* ------------------------------------------------------------------------ */

/* Reflection x = 2 min(u, 1-u) is exact (1-u exact for u >= 1/2, Sterbenz);
   v = -log x; sign by u - 1/2 (+0 at u = 1/2).  u = 0 -> -inf, u = 1 -> +inf,
   u outside [0,1] or NaN -> NaN (Section 7.2 reflection; the paper's kernels
   leave u in {0,1} to NaN). */
__device__ __forceinline__ double reflect(double u) { return __builtin_fmin(u, 1.0 - u); }

__device__ __forceinline__ double quantile_v(double u)
{
    const double p = reflect(u);
    return neg_log_unit(p + p);
}

/* mag is finite where p = min(u, 1-u) = 0; p < 0 outside [0,1].  The specials
   are added, with one 32-bit select each: an inf or NaN for p = 0, p < 0 or
   NaN, 0 otherwise. */
__device__ __forceinline__ double quantile_finish(double u, double mag)
{
    const double p = reflect(u);
    int special = p == 0.0 ? 0x7ff00000 : 0x7ff80000;
    special = p > 0.0 ? 0 : special;
    return __builtin_copysign(mag + __hiloint2double(special, 0), u - 0.5);
}

/* The exponential-coordinate path for any u (plain mode): v = -log(2 min(u,
   1-u)), Q(v), sign and specials. */
__device__ __forceinline__ double outer_quantile_f64(double u)
{
    const OuterPtr c = outer_ptr();
    const double p = reflect(u);
    return quantile_finish(u, expcoord_q_plain(neg_log_unit(p + p, c->log_r), c));
}

/* Central piece, |q| <= 0.45 with q = u - 1/2 (90% of uniform draws):
   w = q P8(r)/Q8(r), r = 0.2025 - q^2, relative error 6e-17 after rounding;
   no logarithm.  q is exact for u >= 1/4 and within half an ulp below, which
   moves w by at most 2.3e-16 relative at |q| = 0.45.  Other q give
   unspecified values. */
__device__ __forceinline__ bool is_central(double q) { return __builtin_fabs(q) <= QM_CENTRAL_QMAX; }

__device__ __forceinline__ double central_quantile(double q)
{
    double r = __builtin_fma(-q, q, QM_CENTRAL_X);
    return div_pos(q * horner(r, QM_CENTRAL_P), horner(r, QM_CENTRAL_Q));
}

/*
 * FP64 w(u).  Paper mode: the (13,13) rational of Appendix B in the
 * exponential coordinate for every u.  Plain mode: the hybrid of
 * Section 7.3 / Appendix C -- a central piece where most samples fall, the
 * branchless exponential-coordinate path elsewhere -- with the paper's T2
 * central variable (chosen there for a fast single-precision-grade rsqrt)
 * replaced by q itself, which needs no transcendental at all.  Lanes
 * outside the centre take the outer path by wave vote here; the streaming
 * kernel instead gathers them across the wave (k_hybrid), with the
 * same arithmetic per element.
 */
template <bool PAPER>
__device__ __forceinline__ double normal_quantile_f64(double u)
{
    if (PAPER) return quantile_finish(u, expcoord_q_paper(quantile_v(u)));
    double q = u - 0.5;
    bool central = is_central(q);           /* NaN: false */
    double w = central_quantile(q);
    if (wave_any(!central)) {
        double wo = outer_quantile_f64(u);
        w = select_f64(central, w, wo);
    }
    return w;
}

/* 1/sqrt(x) for positive normal x, within about an ulp: the hardware
   reciprocal square root y (~5e-8), then y (1 + e/2 + 3e^2/8) with
   e = 1 - x y^2 (second-order Newton; e is exact up to the rounding of x y).
   Zero, denormal, negative or NaN x give values that callers must not use. */
__device__ __forceinline__ double rsqrt_pos(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    double h = x * y;
    double e = __builtin_fma(-h, y, 1.0);
    double c = __builtin_fma(0.375, e, 0.5);
    return __builtin_fma(y * e, c, y);
}

/*
 * The paper's own FP64 hybrid (Section 7.3, Appendix C), constants as
 * printed.  Every lane forms the T2 coordinate v = |u - 1/2| / sqrt(u(1-u));
 * if v < 15.5 on every lane of the wave, the wave takes Psi(v) = v P14/Q15,
 * otherwise the whole wave takes the branchless (13,13) path of Appendix B.
 * u(1-u) is formed as a product rather than the printed u - u*u, which
 * cancels near u = 1 (relative error up to 5e-14 at u = 0.999 there, 1.5
 * ulp here).  u = 1/2 -> +0; u = 0, 1, NaN or outside [0,1] give v >= 15.5
 * or NaN, so the branchless path's specials apply.
 */
__device__ __forceinline__ double t2_coord(double u, double& q)
{
    q = u - 0.5;
    return __builtin_fabs(q) * rsqrt_pos(u * (1.0 - u));
}

__device__ __forceinline__ double t2_psi(double v, double q)
{
    return __builtin_copysign(div_pos(v * horner(v, QM_PAPER_T2_P14), horner(v, QM_PAPER_T2_Q15)), q);
}

__device__ __forceinline__ double normal_quantile_f64_t2(double u)
{
    double q;
    double v = t2_coord(u, q);
    if (__all((int)(v < QM_PAPER_T2_VMAX))) return t2_psi(v, q);
    return quantile_finish(u, expcoord_q_paper(quantile_v(u)));
}

/* Exponential -> normal, FP64: v = |x| directly, odd extension.  Paper mode
   takes the (13,13) rational whatever v.  Plain mode splits into that
   rational (_main) and, for v > 42, the deep-tail piece and what lies beyond
   it (_rare, entered by wave vote), so that a lane's elements can share one
   vote; NaN and inf are rare too. */
__device__ __forceinline__ double exp_to_normal_f64_paper(double x)
{
    double v = __builtin_fabs(x);
    double mag = expcoord_q_paper(v);
    mag = (v == __builtin_inf()) ? v : mag;
    return __builtin_copysign(mag, x);
}

__device__ __forceinline__ double exp_to_normal_f64_main(double x, bool* rare)
{
    const double v = __builtin_fabs(x);
    *rare = !(v <= QM_TAIL_VMIN);
    return __builtin_copysign(div_pos(v * horner(v, QM_PAPER_P13), horner(v, QM_PAPER_Q13)), x);
}

__device__ __forceinline__ double exp_to_normal_f64_rare(double x)
{
    const double v = __builtin_fabs(x);
    const double s = sqrt_pos(v);
    double q = div_pos(s * horner(s, QM_TAIL_P), horner(s, QM_TAIL_Q));
    const bool far = v > QM_TAIL_VMAX && v < __builtin_inf();
    if (wave_any(far)) {
        const double f = expcoord_far(far ? v : 1000.0);
        q = far ? f : q;
    }
    q = (v == __builtin_inf()) ? v : q;
    return __builtin_copysign(q, x);
}

/* ------------------------------------------------------------------------ */
/* FP32 + FP64-refine form.                                                  */
/* ------------------------------------------------------------------------ */

/* -log(x) for x in (0, 1] in FP32 with the hardware log2, denormals scaled
   into the normal range first (accuracy is only needed at the seed level). */
__device__ __forceinline__ float neg_log_f32(float x)
{
    const float LN2F = 0.693147180559945309f;
    bool sub = x < 0x1p-126f;
    float xs = sub ? x * 0x1p32f : x;
    float l2 = __builtin_amdgcn_logf(xs);          /* v_log_f32: log2 */
    return __builtin_fmaf(-l2, LN2F, sub ? 32.0f * LN2F : 0.0f);
}

/* a / b to ~3e-15 for positive b of moderate size: hardware reciprocal and
   one Newton step, no residual correction (enough before a rounding to
   FP32). */
__device__ __forceinline__ double div_pos_fast(double a, double b)
{
    double y = __builtin_amdgcn_rcp(b);
    double e = __builtin_fma(-b, y, 1.0);
    y = __builtin_fma(e, y, y);
    return a * y;
}

/*
 * The FP32+refine form: FP32 in and out, every step in FP64, rounded once.
 * FP64 fused multiply-adds issue at the FP32 rate on gfx950 (4.4-5 cycles a
 * wave against 4.2, packed FP32 off), so what counts is their number, and a
 * rational fitted to the accuracy that the rounding leaves room for takes
 * fewer than an FP32 seed with an FP64 correction step against erf or erfc,
 * which evaluates two or three functions for one: 21 issue slots against 28
 * for the central piece, 44 against 71 for the outer one, 37 against 69 for
 * exponential -> normal.  Before the rounding the central piece is off by
 * 2.8e-9 relative at most, the outer one by 6e-10 and exponential -> normal
 * by 6e-14, nowhere more than a seed and correction step were in the same
 * range: those had 4.8e-9 to 2.3e-8, 1.0e-9 (|z| between 4 and 5) to 1.0e-8,
 * and 1.5e-13 (between 5 and 10) or more; rationals of one or two degrees
 * less, outer 3e-9, exponential -> normal 9.5e-12, were further off in parts
 * of their ranges.  MI355X, per pass, without the later
 * steps: 2^24 exponential -> normal 39.4 -> 29.0
 * us, 2^26 mixture quantiles 106 -> 102, 2^26 fused quantiles 98.3 -> 94.4
 * (all bound by vector instructions before).
 */

/* Phi^{-1}(u) for FP32 u outside the centre: p = min(u, 1-u) (exact), v =
   -log 2p from p = m 2^e (7.1e-10, a third of that in z), Q(v) = P7/Q7. */
__device__ __forceinline__ float outer_quantile_f32(float u)
{
    const double LN2 = 0.69314718055994530942;
    const float om = 1.0f - u;                  /* exact for u >= 1/2 */
    const float p = (u < om) ? u : om;
    const double pd = (double)p;                /* FP32 denormals are normal here */
    const double m = __builtin_amdgcn_frexp_mant(pd);
    const int e = __builtin_amdgcn_frexp_exp(pd);
    const OuterPtr c = outer_ptr();
    const double v = __builtin_fma((double)~e, LN2, -horner(m - 0.75, c->log32));   /* ~e = -1 - e */
    float mag = (float)div_pos_fast(horner(v, c->p32), horner(v, c->q32));
    /* u = 0 and u = 1 both give p = 0: +-inf by the sign of u - 1/2; NaN and
       u outside [0, 1] give NaN */
    mag = p > 0.0f ? mag : p == 0.0f ? __builtin_inff() : __builtin_nanf("");
    return __builtin_copysignf(mag, u - 0.5f);
}

/* Central piece of the FP32+refine form, |q| <= 0.45, q = u - 1/2 (exact in
   FP64 for FP32 u): q P4(r)/Q4(r), r = 0.2025 - q^2. */
__device__ __forceinline__ float central_quantile_f32(double q)
{
    const double r = __builtin_fma(-q, q, QM_CENTRAL_X);
    return (float)div_pos_fast(q * horner(r, QM_D32_CP), horner(r, QM_D32_CQ));
}

/* Phi^{-1}(u) for FP32 u, FP32+refine form: the hybrid of the FP64 path
   (central piece; the outer path by wave vote here, gathered across the
   wave by the streaming kernel, with the same arithmetic per element). */
__device__ __forceinline__ float normal_quantile_f32_refine(float u)
{
    double qd = (double)u - 0.5;
    bool central = is_central(qd);          /* NaN: false */
    float w = central_quantile_f32(qd);
    if (wave_any(!central)) {
        float wo = outer_quantile_f32(u);
        w = central ? w : wo;
    }
    return w;
}

/* Phi^{-1}(u), FP32 u, paper's (5,6) in FP32 verbatim (Appendix A), with the
   specials fixed as above. */
__device__ __forceinline__ float normal_quantile_f32_paper(float u)
{
    float om = 1.0f - u;
    float p = (u < om) ? u : om;
    float v = neg_log_f32(p + p);
    float mag = v * hornerf(v, QM_PAPER_P5) * __builtin_amdgcn_rcpf(hornerf(v, QM_PAPER_Q6));
    float w = __builtin_copysignf(mag, u - 0.5f);
    w = (u == 0.0f) ? -__builtin_inff() : w;
    w = (u == 1.0f) ? __builtin_inff() : w;
    w = (u >= 0.0f && u <= 1.0f) ? w : __builtin_nanf("");
    return w;
}

/* Phi^{-1}(u), FP32 u, evaluated by the plain FP64 path and rounded. */
__device__ __forceinline__ float normal_quantile_f32_plain(float u)
{
    return (float)normal_quantile_f64<false>((double)u);
}

/* Exponential -> normal for FP32 x: Q(v) = v P12(v)/Q12(v), v = |x| <= 103;
   beyond (also inf and NaN) the plain FP64 map, rounded. */
__device__ __forceinline__ float exp_to_normal_f32_main(float x, bool* rare)
{
    const float v = __builtin_fabsf(x);
    *rare = !(v <= 103.0f);
    const double vd = (double)v;
    return __builtin_copysignf((float)div_pos_fast(vd * horner(vd, QM_E32_P), horner(vd, QM_E32_Q)), x);
}

/* The FP64 map of any x, out of line. */
__device__ __noinline__ double exp_to_normal_f64_whole(double x)
{
    bool rare;
    double z = exp_to_normal_f64_main(x, &rare);
    if (wave_any(rare)) {
        const double r = exp_to_normal_f64_rare(x);
        z = rare ? r : z;
    }
    return z;
}

__device__ __forceinline__ float exp_to_normal_f32_rare(float x) { return (float)exp_to_normal_f64_whole((double)x); }

}  // namespace qm
