/*
 * qm_batch.hip -- one persistent launch over many requests of mixed kind,
 * dtype, mode and nu.
 *
 * Every request is cut into chunks of hdr->chunk elements; chunks are numbered
 * globally in request order (chunk_base = prefix sum).  Each workgroup
 * repeatedly claims the next chunk from a device counter, finds its request
 * by binary search over chunk_base, and evaluates it with the same
 * per-element functions as the single-request kernels, so every output is
 * bitwise identical to the single call's.  A chunk belongs to one request,
 * so the kind switch and the wave votes inside the maps are uniform across
 * the workgroup.  A Student t or hyperbolic chunk stages its table in LDS
 * unless the workgroup's previous chunk already did.  The loop ends when the counter
 * passes the last chunk, which every workgroup reaches without waiting on
 * any other.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "qm_batch.h"
#include "qm_device.hpp"
#include "qm_hybrid.hpp"
#include "qm_hyp_device.hpp"
#include "qm_student_device.hpp"

namespace qm {

/* 16-byte vectors per lane, BATCH_UNROLL rows in flight per wave (two
   doubles or four floats each), as the streaming kernels read them. */
constexpr int BATCH_UNROLL = 2;

/* Elements [begin, end) of one request by the whole workgroup, walked by
   its four waves as the single-request kernels walk an array. */
template <typename T, class Map>
__device__ __forceinline__ void chunk_walk(const void* in, void* out, uint64_t begin, uint64_t end, const Map& map)
{
    const Span<T> s = make_span((const T*)in + begin, (T*)out + begin, end - begin);
    const uint32_t lane = wave_lane();
    Walk<T, BATCH_UNROLL> w;
    w.begin(s, wave_uniform(threadIdx.x >> 6), blockDim.x >> 6, lane);
    w.run(s, lane, map);
    run_edges(s, map);
}

extern __shared__ __attribute__((aligned(16))) double lds_tab[];

/* One chunk per op.  Each is a separate, non-inlined function so that its
   constants and registers are its own: inlined together, the union of all
   maps' loop-invariant constants would crowd the persistent loop. */
template <typename T, class Op>
static __device__ __noinline__ void chunk_op(const void* in, void* out, uint64_t begin, uint64_t end)
{
    chunk_walk<T>(in, out, begin, end, ElementMap<T, Op>());
}

/* LDS list of the hybrid quantiles' gather: 64 K elements per wave (K = 4
   FP64 or 8 FP32 per lane, two 16-byte vectors), 8 KB per workgroup of four
   waves. */
constexpr int GATHER_DOUBLES_PER_WAVE = 64 * 4;

/* Hybrid quantile chunk (FP64 plain, FP32+refine): the streaming kernel's
   gather, so that the outer path runs once per 64 outer elements rather than
   on every lane of a wave holding one; bitwise the per-element function. */
template <typename T, class H>
static __device__ __noinline__ void chunk_hybrid(const void* in, void* out, uint64_t begin, uint64_t end, double* gather)
{
    T* buf = reinterpret_cast<T*>(gather + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * GATHER_DOUBLES_PER_WAVE);
    chunk_walk<T>(in, out, begin, end, HybridMap<T, H>{buf, wave_lane()});
}

/* Student t from the table in LDS (referenced by symbol, so the loads stay
   LDS loads). */
template <typename T, int DEG>
static __device__ __noinline__ void chunk_t(const void* in, void* out, uint64_t begin, uint64_t end,
                                            const StudentParams P)
{
    chunk_walk<T>(in, out, begin, end, StudentMap<T, DEG>{lds_tab, P});
}

/* Exponential -> hyperbolic from the cells in LDS. */
template <typename T, int DEG>
static __device__ __noinline__ void chunk_h(const void* in, void* out, uint64_t begin, uint64_t end, const HypParams H)
{
    chunk_walk<T>(in, out, begin, end, HypMap<T, DEG>{lds_tab, H});
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_batch(BatchHeader* hdr, const BatchReq* __restrict__ reqs)
{
    __shared__ uint64_t s_chunk;
    __shared__ double gather[4 * GATHER_DOUBLES_PER_WAVE];
    const double* loaded = nullptr;        /* table currently in LDS (uniform) */
    const uint64_t total = hdr->total_chunks;
    const uint64_t chunk = hdr->chunk;
    const uint32_t nreq = hdr->nreq;
    uint32_t* const left = hdr->left;
    uint32_t* const done = hdr->done;
    for (;;) {
        if (threadIdx.x == 0) s_chunk = atomicAdd(reinterpret_cast<unsigned long long*>(&hdr->counter), 1ull);
        __syncthreads();
        const uint64_t c = s_chunk;
        __syncthreads();
        if (c >= total) break;
        /* last request with chunk_base <= c (every listed request has chunks) */
        uint32_t lo = 0, hi = nreq - 1;
        while (lo < hi) {
            uint32_t mid = (lo + hi + 1) >> 1;
            if (reqs[mid].chunk_base <= c) lo = mid; else hi = mid - 1;
        }
        const BatchReq& R = reqs[lo];
        const uint64_t begin = (c - R.chunk_base) * chunk;
        const uint64_t end = begin + chunk < R.n ? begin + chunk : R.n;
        switch (R.op) {
        case BOP_NQ64_PLAIN: chunk_hybrid<double, HybridNQ64>(R.in, R.out, begin, end, gather); break;
        case BOP_NQ64_PAPER: chunk_op<double, OpNQ64Paper>(R.in, R.out, begin, end); break;
        case BOP_NQ32_REFINE: chunk_hybrid<float, HybridNQ32>(R.in, R.out, begin, end, gather); break;
        case BOP_NQ32_PAPER: chunk_op<float, OpNQ32Paper>(R.in, R.out, begin, end); break;
        case BOP_NQ32_PLAIN: chunk_op<float, OpNQ32Plain>(R.in, R.out, begin, end); break;
        case BOP_E64_PLAIN: chunk_op<double, OpE64Plain>(R.in, R.out, begin, end); break;
        case BOP_E64_PAPER: chunk_op<double, OpE64Paper>(R.in, R.out, begin, end); break;
        case BOP_E32_REFINE: chunk_op<float, OpE32Refine>(R.in, R.out, begin, end); break;
        case BOP_E32_PLAIN: chunk_op<float, OpE32Plain>(R.in, R.out, begin, end); break;
        case BOP_T64:
        case BOP_T32: {
            if (R.P.identity) {
                if (R.op == BOP_T64) chunk_op<double, OpCopy<double>>(R.in, R.out, begin, end);
                else chunk_op<float, OpCopy<float>>(R.in, R.out, begin, end);
                break;
            }
            if (loaded != R.coef) {
                __syncthreads();
                stage_table(lds_tab, R.coef, R.P);
                __syncthreads();
                loaded = R.coef;
            }
            if (R.op == BOP_T64) {
                if (R.P.row_shift == 4) chunk_t<double, T_DEGREE_HIGH>(R.in, R.out, begin, end, R.P);
                else chunk_t<double, T_DEGREE_LOW>(R.in, R.out, begin, end, R.P);
            }
            else chunk_t<float, T_DEGREE_F32>(R.in, R.out, begin, end, R.P);
            break;
        }
        case BOP_H64:
        case BOP_H32: {
            if (loaded != R.H.r.gcoef) {
                __syncthreads();
                if (R.op == BOP_H64) stage_hyp<HYP_DEGREE>(lds_tab, R.H);
                else stage_hyp<HYP_DEGREE_F32>(lds_tab, R.H);
                __syncthreads();
                loaded = R.H.r.gcoef;
            }
            if (R.op == BOP_H64) chunk_h<double, HYP_DEGREE>(R.in, R.out, begin, end, R.H);
            else chunk_h<float, HYP_DEGREE_F32>(R.in, R.out, begin, end, R.H);
            break;
        }
        default:
            break;
        }
        if (done && R.flagged) {
            /* per-request completion: each thread's stores of the chunk
               reach device scope before the workgroup counts the chunk;
               the workgroup that counts a request's last chunk raises its
               host-visible flag (release at system scope).  Only requests
               of a few chunks are flagged: the fence writes back the L2,
               too dear for every chunk of a large batch */
            __threadfence();
            __syncthreads();
            if (threadIdx.x == 0 &&
                __hip_atomic_fetch_add(left + lo, ~0u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == 1u)
                __hip_atomic_store(done + lo, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

/*
 * Descriptor memory of the allocation-free batch entry point: a header and
 * up to QM_BATCH_NOALLOC_MAX_REQUESTS records, one copy per GPU, held until
 * the process ends.  Host code never passes the array's name to a kernel or
 * a copy (on the host it is only a stand-in for the symbol): it uses the
 * device address that batch_scratch_address looks up once per device.
 */
static __device__ __align__(256) unsigned char scratch[BATCH_SCRATCH_BYTES];

hipError_t batch_scratch_address(int device, void** out)
{
    static std::mutex mu;
    static void* addr[BATCH_SCRATCH_MAX_DEVICES] = {};
    *out = nullptr;
    if (device < 0 || device >= BATCH_SCRATCH_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;   /* the caller makes `device` current */
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = p;
    }
    *out = addr[device];
    return hipSuccess;
}

hipError_t launch_batch(BatchHeader* d_hdr, const BatchReq* d_reqs, size_t lds_bytes, uint64_t blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch, dim3((unsigned)blocks), dim3(256), lds_bytes, s, d_hdr, d_reqs);
    return hipGetLastError();
}

}  // namespace qm
