/*
 * qm_hyp.hip -- exponential -> hyperbolic recycling kernels (Section 8.1).
 *
 * x = mu + sign(v) Q_side(|v|), Q = a R(a), a = |v|, with R the per-cell
 * polynomial of the side (v >= 0: the right map; v < 0: the mirrored left
 * map) built on the host from the recycling ODE (qm_hyp_table.cpp).  Cells
 * are eight per octave of t = 1 + a/v0 (v0 shared by both sides), so the
 * cell index is the exponent and top three mantissa bits of t, and the
 * cell's centre is t with its lower bits replaced: no table search, no
 * per-side selects but a row offset.  Each workgroup stages the cells that
 * reach a = 64 / rate (all but a fraction e^-64 of the base's samples) of
 * both sides in LDS, then streams 16-byte vectors; a lane evaluates all its
 * elements' polynomials (independent chains) before one wave vote admits
 * the rare far elements: the side's further cells from global memory, and
 * from v_top on the large-v form a + c0 + c1/a + c2/a^2 (for variance-gamma
 * targets, whose tail carries a power x^(lambda-1), the form with a log Q
 * term, solved by three fixed-point steps).  The same kernel serves the
 * hyperbolic (Section 8.1) and variance-gamma (Section 8.2) tables.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <algorithm>

#include "qm_hyp_device.hpp"
#include "qm_internal.h"
#include "qm_stream.hpp"

namespace qm {

template <typename T, int UNROLL, int DEG>
__global__ __launch_bounds__(256) void k_hyperbolic(Span<T> s, HypParams P)
{
    extern __shared__ __attribute__((aligned(16))) double lds_hyp[];
    const uint32_t lane = wave_lane();
    Walk<T, UNROLL> w;
    w.begin(s, wave_uniform(blockIdx.x * 4ull + (threadIdx.x >> 6)), gridDim.x * 4ull, lane);
    stage_hyp<DEG>(lds_hyp, P);
    __syncthreads();
    const HypMap<T, DEG> map = {lds_hyp, P};
    w.run(s, lane, map);
    if (blockIdx.x == 0) run_edges(s, map);
}

/* Bytes of LDS per workgroup for the cells: 31 octaves of both sides in FP64,
   within the dynamic LDS of the batch kernel. */
constexpr size_t HYP_LDS_MAX = 55 * 1024;

static bool side_valid(const HypSide& s, int degree, uint64_t ncoef)
{
    return s.degree == degree && s.noct >= 1 && s.noct <= HYP_MAX_OCT && s.ncell == HYP_SUB * s.noct &&
           s.coef_offset + (uint64_t)s.ncell * (degree + 1) <= ncoef && s.v0 > 0 && s.v_top > 0 &&
           (s.origin == 0 || s.origin == 1);
}

/* Octaves of t = 1 + v/v0 that reach 64 / rate. */
static int octaves_to(double v0, double rate)
{
    int k = 1;
    while (k < HYP_MAX_OCT && v0 * ((double)(1ull << k) - 1.0) < 64.0 / rate) ++k;
    return k;
}

static void side_far(const HypSide& s, const double* d_block, HypSideFar* f)
{
    f->v_top = s.v_top;
    f->c0 = s.far_c0;
    f->c1 = s.far_c1;
    f->c2 = s.far_c2;
    f->clog = s.far_clog;
    f->gcoef = d_block + s.coef_offset;
    f->ncell = s.ncell;
}

bool make_hyp_params(const HypTableHeader& h, bool f32, const HypTableHeader* d_table, uint64_t ncoef, double mu,
                     HypParams* P, size_t* lds_bytes)
{
    const HypSide& R = f32 ? h.right32 : h.right;
    const HypSide& L = f32 ? h.left32 : h.left;
    const int deg = f32 ? HYP_DEGREE_F32 : HYP_DEGREE;
    if (!side_valid(R, deg, ncoef) || !side_valid(L, deg, ncoef) || R.v0 != L.v0 || R.inv_v0 != L.inv_v0 ||
        R.origin != L.origin)
        return false;
    const double* d_block = reinterpret_cast<const double*>(reinterpret_cast<const char*>(d_table) + sizeof(HypTableHeader));
    const int stride = f32 ? HypRow<HYP_DEGREE_F32>::lds : HypRow<HYP_DEGREE>::lds;
    /* LDS cells per side: through the octave reaching 64 / rate on either
       side, within both sides' cells and the LDS budget */
    int noct = std::max(octaves_to(R.v0, h.alpha - h.beta), octaves_to(R.v0, h.alpha + h.beta));
    noct = std::min(noct, std::min(R.noct, L.noct));
    noct = std::min(noct, (int)(HYP_LDS_MAX / (2 * stride * sizeof(double) * HYP_SUB)));
    P->v0 = R.v0;
    P->inv_v0 = R.inv_v0;
    P->mu = mu;
    side_far(R, d_block, &P->r);
    side_far(L, d_block, &P->l);
    P->nlds = HYP_SUB * noct;
    P->jlo = R.origin ? HYP_SUB : 0;
    /* the cells, and both sides' origin series */
    *lds_bytes = (size_t)2 * (P->nlds * stride + (R.origin ? deg + 1 : 0)) * sizeof(double);
    return true;
}

template <typename T, int DEG>
static hipError_t launch_h(const void* in, void* out, uint64_t n, const HypParams& P, size_t lds, hipStream_t s,
                           KernelShape shape, int cus)
{
    const Span<T> a = make_span(static_cast<const T*>(in), static_cast<T*>(out), n);
    /* targets with the origin series: a tile's passes over it are a latency
       that two tiles do not hide and more do (variance-gamma 4.25, 2^26 FP64:
       196 us at 64 workgroups per unit, 219 with two tiles each; 2^28 765 and
       853) */
    if (P.jlo) shape.big_blocks = 64 * (uint64_t)cus;
    else fit_to_table(shape, lds, H_TABLE_BLOCKS, cus);
    const int u = launch_unroll(a.nvec, shape, cus);
    const dim3 grid(launch_blocks(a.nvec, u, shape)), block(256);
    with_unroll(u, [&](auto U) {
        hipLaunchKernelGGL((k_hyperbolic<T, decltype(U)::value, DEG>), grid, block, lds, s, a, P);
    });
    return hipGetLastError();
}

hipError_t launch_hyperbolic(int dtype, int mode, const void* in, void* out, uint64_t n, const HypTableHeader* d_table,
                             const HypTableHeader& h, uint64_t ncoef, double mu, hipStream_t s,
                             const LaunchShape& shape)
{
    const bool f32 = dtype == QM_F32 && mode == QM_F32_REFINE;
    if (!f32 && !(dtype == QM_F64 && mode == QM_PLAIN)) return hipErrorInvalidValue;
    HypParams P;
    size_t lds = 0;
    if (!make_hyp_params(h, f32, d_table, ncoef, mu, &P, &lds)) return hipErrorInvalidValue;
    if (f32) return launch_h<float, HYP_DEGREE_F32>(in, out, n, P, lds, s, shape.hyperbolic[0], shape.cus);
    return launch_h<double, HYP_DEGREE>(in, out, n, P, lds, s, shape.hyperbolic[1], shape.cus);
}

}  // namespace qm

/* Host evaluation of the origin series' power (include/qm_debug.h): the
   reciprocal's float rounding stands in for the hardware's 5e-8. */
extern "C" int qm_debug_pow_small(const double* a, double rho, double* w, int n)
{
    for (int i = 0; i < n; ++i) w[i] = qm::pow_small(a[i], rho, [](double x) { return (double)(float)(1.0 / x); });
    return 0;
}
