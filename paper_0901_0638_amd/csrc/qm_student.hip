/*
 * qm_student.hip -- normal -> Student t recycling kernels.
 *
 * t = F_nu^{-1}(Phi(z)) = z R(y), y = z^2, with R the per-cell polynomial
 * built on the host from the recycling ODE (qm_table.cpp).  Each workgroup
 * stages the cells of y <= 100 in LDS once, then streams 16-byte vectors as
 * the other elementwise kernels do.  Per element: the cell index from
 * y = s^2 by one multiply, the offset d = s^2 - y_c by one fused
 * multiply-add (so the full input precision reaches the polynomial: log R
 * grows like y/(2 nu)), the cell's coefficients from LDS, Horner in d, one
 * multiply by z.  FP64 outputs use degree-7 cells where at most 200 of them
 * cover y <= 100 (nu >= 3 or so) and degree-15 cells else, FP32 outputs their
 * own degree-7 cells.  Elements beyond (|z| > 10, probability below 1e-23 for a normal
 * sample) are entered by a wave vote: the table's further cells from global
 * memory, then the two-term tail formula of Section 3.5 in log space.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include "qm_device.hpp"
#include "qm_internal.h"
#include "qm_stream.hpp"
#include "qm_student_device.hpp"

namespace qm {

template <typename T, int UNROLL, int DEG>
__global__ __launch_bounds__(256) void k_student(Span<T> s, StudentParams P)
{
    extern __shared__ __attribute__((aligned(16))) double lds_tab[];
    const uint32_t lane = wave_lane();
    Walk<T, UNROLL> w;
    w.begin(s, wave_uniform(blockIdx.x * 4ull + (threadIdx.x >> 6)), gridDim.x * 4ull, lane);
    stage_table(lds_tab, P.gcoef, P);
    __syncthreads();
    const StudentMap<T, DEG> map = {lds_tab, P};
    w.run(s, lane, map);
    if (blockIdx.x == 0) run_edges(s, map);
}

/* nu = +inf: the identity map (Section 3.1, n -> infinity gives Q = z). */
template <typename T>
__global__ __launch_bounds__(256) void k_identity(const T* in, T* out, uint64_t n)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) out[i] = in[i];
}

/* LDS row stride in doubles for nlds rows of `row` coefficients: even, so
   that every row starts on a 16-byte boundary and is read in 16-byte pieces,
   and an odd number of 16-byte groups, so that the rows start in all of them:
   10 for rows of 8, 18 for rows of 16 (nu = 1, 2^22 elements: 14.2 us on
   MI355X, 14.8 with rows of 16) while that leaves room in 64 KB for the
   fused generator's gather list, else 16 (the widest sets take 480 rows).
   QM_T_LDS_STRIDE (16..24) and QM_T8_LDS_STRIDE (8..24), even values only,
   override them (tuning). */
static int stride_from_env(const char* name, int row)
{
    const char* e = getenv(name);
    const int v = e ? atoi(e) : 0;
    return (v >= row && v <= 24 && v % 2 == 0) ? v : 0;
}

static int student_lds_stride(int row, int nlds)
{
    static const int e16 = stride_from_env("QM_T_LDS_STRIDE", T_DEGREE_HIGH + 1);
    static const int e8 = stride_from_env("QM_T8_LDS_STRIDE", T_DEGREE_LOW + 1);
    if (row != T_DEGREE_HIGH + 1) return e8 ? e8 : row + 2;
    if (e16) return e16;
    return (size_t)nlds * (row + 2) * sizeof(double) <= 48 * 1024 ? row + 2 : row;
}

static bool cells_valid(const TCells& c, int degree)
{
    return c.degree == degree && c.stride == degree + 1 && c.nlds >= 1 && c.ncell >= c.nlds;
}

/* Every row of the table's LDS range (|z| <= 10) is staged.  Half of it (|z| <=
   7, all but 2.6e-12 of normal draws) is 0 to 2% faster on normal draws (MI355X,
   2^26 FP64, nu = 1: 170.7 us against 174.4; nu = 30 169.3 and 169.0), but
   inputs that do reach 7 < |z| <= 10 then go one element of each lane at a
   time through the far path (uniform on +-10, nu = 4: 284 against 179). */
StudentParams make_params(const TTableHeader& h, const TCells& c, const double* d_rows)
{
    StudentParams P;
    P.h = c.h;
    P.inv_h = c.inv_h;
    P.centre_offset = c.centre_offset;
    P.y_max = c.y_max;
    P.gcoef = d_rows;
    P.log_K = h.log_K;
    P.tail_a = h.tail_a[0];
    P.sqrt_nu = __builtin_sqrt(h.nu);
    P.nu = h.nu;
    P.ncell = c.ncell;
    P.nlds = c.nlds;              /* 0 for nu = +inf, which has no cells */
    P.y_lds = c.y_lds;
    P.identity = h.identity;
    P.row_shift = c.stride == 16 ? 4 : 3;
    P.lds_stride = student_lds_stride(c.stride, P.nlds);
    return P;
}

template <typename T, int DEG>
static hipError_t launch_t(const void* in, void* out, uint64_t n, const double* d_block, const TTableHeader& h,
                           hipStream_t s, const LaunchShape& shape_all)
{
    KernelShape shape = shape_all.student[sizeof(T) == 8];
    if (h.identity) {
        uint64_t blocks = (n + 255) / 256;
        if (blocks > shape.max_blocks) blocks = shape.max_blocks;
        hipLaunchKernelGGL((k_identity<T>), dim3((unsigned)blocks), dim3(256), 0, s,
                           static_cast<const T*>(in), static_cast<T*>(out), n);
        return hipGetLastError();
    }
    const TCells& c = sizeof(T) == 8 ? h.f64 : h.f32;
    const StudentParams P = make_params(h, c, d_block + c.coef_offset);
    const size_t lds = student_lds_bytes(P);
    if (lds > 65536) return hipErrorInvalidValue;   /* beyond the dynamic LDS a launch may ask for */
    fit_to_table(shape, lds, T_TABLE_BLOCKS, shape_all.cus);
    if (DEG == T_DEGREE_HIGH) {
        /* rows of 16: two tiles from 2^26 elements on (2^25, nu = 1: 91 to 98 us
           on two cards, 89 to 92 on the fixed grid; 2^26 174, 179 to 191), one
           only where a thread stages one piece (2^28: 694 us with 32 rows, 761
           with 33) */
        shape.big_vecs *= 2;
        if (P.nlds > 32) shape.huge_vecs = 0;
    }
    const Span<T> a = make_span(static_cast<const T*>(in), static_cast<T*>(out), n);
    const int u = launch_unroll(a.nvec, shape, shape_all.cus);
    const dim3 grid(launch_blocks(a.nvec, u, shape)), block(256);
    with_unroll(u, [&](auto U) {
        hipLaunchKernelGGL((k_student<T, decltype(U)::value, DEG>), grid, block, lds, s, a, P);
    });
    return hipGetLastError();
}

hipError_t launch_student(int dtype, int mode, const void* in, void* out, uint64_t n,
                          const TTableHeader* d_table, const TTableHeader& h_table,
                          hipStream_t s, const LaunchShape& shape)
{
    if (!h_table.identity && !((cells_valid(h_table.f64, T_DEGREE_LOW) || cells_valid(h_table.f64, T_DEGREE_HIGH)) &&
                               cells_valid(h_table.f32, T_DEGREE_F32)))
        return hipErrorInvalidValue;
    const double* d_block = table_block(d_table);
    if (dtype == QM_F64 && mode == QM_PLAIN) {
        if (h_table.identity || h_table.f64.degree == T_DEGREE_LOW)
            return launch_t<double, T_DEGREE_LOW>(in, out, n, d_block, h_table, s, shape);
        return launch_t<double, T_DEGREE_HIGH>(in, out, n, d_block, h_table, s, shape);
    }
    if (dtype == QM_F32 && mode == QM_F32_REFINE)
        return launch_t<float, T_DEGREE_F32>(in, out, n, d_block, h_table, s, shape);
    return hipErrorInvalidValue;
}

}  // namespace qm

/* What a launch stages of the table for nu (include/qm_debug.h). */
extern "C" int qm_debug_student_staging(double nu, int f32, double* y_staged, unsigned long long* lds_bytes)
{
    qm::HostTTable t{};
    char err[256] = {0};
    if (qm::build_student_table(nu, &t, err, sizeof err) != 0) return -1;
    const qm::StudentParams P = qm::make_params(t.hdr, f32 ? t.hdr.f32 : t.hdr.f64, nullptr);
    qm::free_student_table(&t);
    *y_staged = P.y_lds;
    *lds_bytes = P.identity ? 0 : qm::student_lds_bytes(P);
    return P.nlds;
}
