/*
 * qm_internal.h -- declarations shared by the library's translation units
 * (not part of the public ABI).
 */
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/qm.h"
#include "qm_hyp_table.h"
#include "qm_table.h"

namespace qm {

/* Launch geometry of one kernel family: at most max_blocks workgroups of
   256, each lane keeping `unroll` 16-byte vectors in flight (1, 2 or 4).
   Launches of big_vecs vectors and more keep big_unroll in flight, with two
   tiles to a workgroup, those of huge_vecs and more four, with one tile (0:
   never); both have at most big_blocks workgroups.  fixed_unroll: `unroll`
   holds for launches of every size. */
struct KernelShape {
    uint64_t max_blocks;
    int unroll, big_unroll;
    bool fixed_unroll;
    uint64_t big_vecs, huge_vecs, big_blocks;
};

/* Per family, measured on MI355X (launch-shape sweeps over 1..1024
   workgroups per CU x 1..4 vectors, 2^17 to 2^29 elements): kernels that
   stage a table run best from few workgroups, the others from many; arrays
   beyond the last-level cache from one for every tile or two. */
struct LaunchShape {
    KernelShape stream;      /* k_map, FP64: exp -> normal, the paper's quantiles */
    KernelShape stream32;    /* k_map, FP32: exp -> normal */
    KernelShape light[2];    /* k_map, [0] FP32: paper and plain quantiles, [1] FP64: the paper's exp -> normal */
    KernelShape hybrid[2];   /* [0] FP32+refine, [1] FP64 quantile: k_hybrid */
    KernelShape uniform[2];  /* [0] FP32, [1] FP64 outputs: k_generate of the uniforms */
    KernelShape generate[2]; /* ... of quantiles */
    KernelShape generate_t[2]; /* ... k_generate_t */
    KernelShape generate_h[2]; /* ... k_generate_h */
    KernelShape student[2];  /* [0] FP32, [1] FP64 outputs: k_student */
    KernelShape hyperbolic[2]; /* [0] FP32, [1] FP64: k_hyperbolic */
    int cus;                 /* compute units of the device */
    int compact;             /* quantiles: gather non-central lanes across the wave */
};

/* Elementwise normal quantile / exp -> normal on one stream. */
hipError_t launch_elementwise(int kind, int dtype, int mode, const void* in, void* out, uint64_t n,
                              hipStream_t s, const LaunchShape& shape);

/* Fused Philox4x32-10 generation and transform (qm_generate.hip). */
hipError_t launch_generate(int kind, int dtype, int mode, uint32_t seed, uint32_t stream, uint64_t first,
                           void* out, uint64_t n, hipStream_t s, const LaunchShape& shape);

/* Fused generation chains (qm_generate.hip): the Student t of the normal
   quantile of each uniform, and the hyperbolic map of each uniform's
   two-sided exponential base sample. */
hipError_t launch_generate_student(int dtype, int mode, uint32_t seed, uint32_t stream, uint64_t first, void* out,
                                   uint64_t n, const TTableHeader* d_table, const TTableHeader& h, hipStream_t s,
                                   const LaunchShape& shape);
hipError_t launch_generate_hyperbolic(int dtype, int mode, uint32_t seed, uint32_t stream, uint64_t first, void* out,
                                      uint64_t n, const HypTableHeader* d_table, const HypTableHeader& h,
                                      uint64_t ncoef, double mu, hipStream_t s, const LaunchShape& shape);

/* The coefficient block that follows a device table's header. */
inline const double* table_block(const TTableHeader* d_table)
{
    return reinterpret_cast<const double*>(reinterpret_cast<const char*>(d_table) + sizeof(TTableHeader));
}

/* Launch the Student t map with a device table (qm_student.hip): FP64
   outputs use the table's f64 cells, FP32 outputs its f32 cells. */
hipError_t launch_student(int dtype, int mode, const void* in, void* out, uint64_t n,
                          const TTableHeader* d_table, const TTableHeader& h_table,
                          hipStream_t s, const LaunchShape& shape);

/* Launch the exponential -> hyperbolic map with a device table
   (qm_hyp.hip); ncoef doubles follow the header. */
hipError_t launch_hyperbolic(int dtype, int mode, const void* in, void* out, uint64_t n, const HypTableHeader* d_table,
                             const HypTableHeader& h, uint64_t ncoef, double mu, hipStream_t s,
                             const LaunchShape& shape);

}  // namespace qm
