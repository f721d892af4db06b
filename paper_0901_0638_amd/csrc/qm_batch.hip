/*
 * qm_batch.hip -- one launch over many requests of mixed kind,
 * dtype, mode and nu.
 *
 * Every request is cut into chunks of a number of elements that its batch
 * sets (batch_chunk in qm_serve.cpp); chunks are numbered globally in
 * request order (chunk_base = prefix sum).  Each workgroup starts with the
 * chunk of its own index and goes on in steps of the grid, finds each
 * chunk's request by its chunk_base, and evaluates it with the same walk and
 * per-element functions as the single-request kernels, so every output is
 * bitwise identical to the single call's.  A chunk belongs to one request,
 * so the kind switch and the wave votes inside the maps are uniform across
 * the workgroup.  A Student t or hyperbolic chunk stages its table in LDS
 * unless the workgroup's previous chunk already did.  Every workgroup reaches
 * the end of its loop without waiting on another.
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

/* Descriptors are read through the constant address space: uniform loads
   into scalar registers, of memory that no launch writes while it runs. */
typedef const __attribute__((address_space(4))) BatchReq* ReqPtr;

__device__ __forceinline__ ReqPtr uniform_req(uint64_t addr)
{
    return (ReqPtr)wave_uniform(addr);
}

/* Part `part` of the `parts` of the request at `addr`, by the whole workgroup.
   The parts' waves take the request's tiles in turn, as the workgroups of a
   single-request launch do; the first part has the edge elements.  Parts that
   were runs of neighbouring tiles read and wrote as many windows as there are
   workgroups, each far from the next (512 requests of 2^10..2^20 elements:
   169.7 us a pass, 166.0 in turn; 4096 of 2^10..2^22: 5.09 ms and 4.97). */
template <typename T, class Map>
__device__ __forceinline__ void chunk_walk(uint64_t addr, uint64_t part, uint64_t parts, const Map& map)
{
    const ReqPtr R = uniform_req(addr);
    part = wave_uniform(part);
    parts = wave_uniform(parts);
    const Span<T> s = make_span((const T*)R->in, (T*)R->out, R->n);
    const uint32_t lane = wave_lane();
    Walk<T, BATCH_UNROLL> w;
    w.begin(s, part * 4 + wave_uniform(threadIdx.x >> 6), parts * 4, lane);
    w.run(s, lane, map);
    if (part == 0) run_edges(s, map);
}

extern __shared__ __attribute__((aligned(16))) double lds_tab[];

/* One chunk per op.  Each is a separate, non-inlined function so that its
   constants and registers are its own: inlined together, the union of all
   maps' loop-invariant constants would crowd the chunk loop.  A request's
   table parameters are read from its descriptor inside (passed by value they
   went through every lane's scratch memory). */
template <typename T, class Op>
static __device__ __noinline__ void chunk_op(uint64_t addr, uint64_t part, uint64_t parts)
{
    chunk_walk<T>(addr, part, parts, typename MapOf<T, Op>::type());
}

/* LDS list of the hybrid quantiles' gather: 64 K elements per wave (K = 4
   FP64 or 8 FP32 per lane, two 16-byte vectors), 8 KB per workgroup of four
   waves. */
constexpr int GATHER_DOUBLES_PER_WAVE = 64 * 4;
__device__ __forceinline__ double* gather_list()
{
    static __shared__ double gather[4 * GATHER_DOUBLES_PER_WAVE];
    return gather + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * GATHER_DOUBLES_PER_WAVE;
}

/* Hybrid quantile chunk (FP64 plain, FP32+refine): the streaming kernel's
   gather, so that the outer path runs once per 64 outer elements rather than
   on every lane of a wave holding one; bitwise the per-element function. */
template <typename T, class H>
static __device__ __noinline__ void chunk_hybrid(uint64_t addr, uint64_t part, uint64_t parts)
{
    chunk_walk<T>(addr, part, parts, HybridMap<T, H>{reinterpret_cast<T*>(gather_list()), wave_lane()});
}

/* Student t from the table in LDS (referenced by symbol, so the loads stay
   LDS loads). */
template <typename T, int DEG>
static __device__ __noinline__ void chunk_t(uint64_t addr, uint64_t part, uint64_t parts)
{
    const StudentParams P = *(const StudentParams*)&uniform_req(addr)->P;
    chunk_walk<T>(addr, part, parts, StudentMap<T, DEG>{lds_tab, P});
}

/* Exponential -> hyperbolic from the cells in LDS. */
template <typename T, int DEG>
static __device__ __noinline__ void chunk_h(uint64_t addr, uint64_t part, uint64_t parts)
{
    const HypParams H = *(const HypParams*)&uniform_req(addr)->H;
    chunk_walk<T>(addr, part, parts, HypMap<T, DEG>{lds_tab, H});
}

/* Part `part` of the `parts` of the request R; *loaded: the table in LDS. */
__device__ __forceinline__ void do_chunk(ReqPtr R, uint64_t part, uint64_t parts, const double** loaded)
{
    const uint64_t addr = (uint64_t)R;
    const uint32_t op = R->op;
    if (op == BOP_T64 || op == BOP_T32) {
        const StudentParams P = *(const StudentParams*)&R->P;
        if (!P.identity && *loaded != P.gcoef) {
            stage_table(lds_tab, P.gcoef, P);
            __syncthreads();
            *loaded = P.gcoef;
        }
    } else if (op == BOP_H64 || op == BOP_H32) {
        const HypParams H = *(const HypParams*)&R->H;
        if (*loaded != H.r.gcoef) {
            if (op == BOP_H64) stage_hyp<HYP_DEGREE>(lds_tab, H);
            else stage_hyp<HYP_DEGREE_F32>(lds_tab, H);
            __syncthreads();
            *loaded = H.r.gcoef;
        }
    }
    switch (op) {
    case BOP_NQ64_PLAIN: chunk_hybrid<double, HybridNQ64>(addr, part, parts); break;
    case BOP_NQ64_PAPER: chunk_op<double, OpNQ64Paper>(addr, part, parts); break;
    case BOP_NQ32_REFINE: chunk_hybrid<float, HybridNQ32>(addr, part, parts); break;
    case BOP_NQ32_PAPER: chunk_op<float, OpNQ32Paper>(addr, part, parts); break;
    case BOP_NQ32_PLAIN: chunk_op<float, OpNQ32Plain>(addr, part, parts); break;
    case BOP_E64_PLAIN: chunk_op<double, OpE64Plain>(addr, part, parts); break;
    case BOP_E64_PAPER: chunk_op<double, OpE64Paper>(addr, part, parts); break;
    case BOP_E32_REFINE: chunk_op<float, OpE32Refine>(addr, part, parts); break;
    case BOP_E32_PLAIN: chunk_op<float, OpE32Plain>(addr, part, parts); break;
    case BOP_T64:
        if (R->P.identity) chunk_op<double, OpCopy<double>>(addr, part, parts);
        else if (R->P.row_shift == 4) chunk_t<double, T_DEGREE_HIGH>(addr, part, parts);
        else chunk_t<double, T_DEGREE_LOW>(addr, part, parts);
        break;
    case BOP_T32:
        if (R->P.identity) chunk_op<float, OpCopy<float>>(addr, part, parts);
        else chunk_t<float, T_DEGREE_F32>(addr, part, parts);
        break;
    case BOP_H64: chunk_h<double, HYP_DEGREE>(addr, part, parts); break;
    case BOP_H32: chunk_h<float, HYP_DEGREE_F32>(addr, part, parts); break;
    default: break;
    }
}

/*
 * A workgroup's chunks: that of its own index and every gridDim.x-th after
 * it.  (Claimed from a device counter, the claims are a serial chain through
 * one memory word: 12 ns each on an idle MI355X and 58 beside the streams, so
 * that 4600 claims took as long as their chunks' work and smaller chunks only
 * more; 512 requests of 2^10..2^20 elements: 270 us a pass with claims, 186
 * without, in smaller chunks.)  The request of a chunk is the last one with chunk_base <= c
 * (every listed request has chunks), found 64 candidates at a time, one per
 * lane: two dependent loads for 4096 requests where a binary search took
 * twelve.
 */
__device__ __forceinline__ void batch_chunks(uint64_t total, uint32_t nreq, ReqPtr reqs, uint32_t* count, uint32_t* done)
{
    const uint32_t lane = wave_lane();
    const double* loaded = nullptr;        /* table currently in LDS (uniform) */
    for (uint64_t c = blockIdx.x; c < total; c += gridDim.x) {
        uint32_t lo = 0, len = nreq;
        while (len > 1) {
            const uint32_t stride = (len + 63) >> 6, i = lane * stride;
            const bool le = i < len && reqs[lo + i].chunk_base <= c;
            const uint32_t skip = ((uint32_t)__popcll(__ballot(le)) - 1) * stride;
            lo += skip;
            len = min(stride, len - skip);
        }
        const ReqPtr R = reqs + lo;
        const uint64_t first = R->chunk_base, next = lo + 1 < nreq ? reqs[lo + 1].chunk_base : total;
        if (c != blockIdx.x) __syncthreads();      /* every wave is done with the LDS */
        do_chunk(R, c - first, next - first, &loaded);
        if (done && R->flagged) {
            /* per-request completion: every wave's stores of the chunk have
               reached the XCD's L2 before the barrier, one thread's release
               then writes that back and counts the chunk; the workgroup
               that counts a request's last chunk raises its host-visible
               flag (release at system scope) */
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (threadIdx.x == 0) {
                __threadfence();
                if (__hip_atomic_fetch_add(count + lo, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
                    R->flagged) {
                    __hip_atomic_store(count + lo, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(done + lo, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_batch(const BatchHeader* hdr, const BatchReq* reqs)
{
    typedef const __attribute__((address_space(4))) BatchHeader* HdrPtr;
    const HdrPtr h = (HdrPtr)(uint64_t)hdr;
    batch_chunks(h->total_chunks, h->nreq, (ReqPtr)(uint64_t)reqs, h->count, h->done);
}

/* The batch in the kernel's arguments: read from the argument segment, which
   starts with them (indexing the parameter would copy it to scratch).  Such a
   batch has no completion flags. */
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_batch_args(BatchArgs)
{
    typedef const __attribute__((address_space(4))) BatchArgs* ArgsPtr;
    const ArgsPtr a = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    batch_chunks(a->h.total_chunks, a->h.nreq, a->r, nullptr, nullptr);
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

hipError_t launch_batch(const BatchHeader* d_hdr, const BatchReq* d_reqs, size_t lds_bytes, uint64_t blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch, dim3((unsigned)blocks), dim3(256), lds_bytes, s, d_hdr, d_reqs);
    return hipGetLastError();
}

/* The descriptors' upload as a kernel that reads the pinned staging memory: a
   copy command goes through another queue, whose hand-over and back cost more
   than the copy (512 requests, 98 KB, MI355X: 180.9 us a pass with the copy
   command, 169.5 with this). */
__global__ __launch_bounds__(256) void k_upload(const uint64_t* host, uint64_t* dev, uint32_t n)
{
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) dev[i] = host[i];
}

hipError_t launch_upload(const void* host, void* dev, size_t bytes, hipStream_t s)
{
    const uint32_t n = (uint32_t)(bytes / 8);
    hipLaunchKernelGGL(k_upload, dim3((n + 255) / 256), dim3(256), 0, s, static_cast<const uint64_t*>(host),
                       static_cast<uint64_t*>(dev), n);
    return hipGetLastError();
}

hipError_t launch_batch_args(const BatchArgs& args, size_t lds_bytes, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_args, dim3((unsigned)args.h.total_chunks), dim3(256), lds_bytes, s, args);
    return hipGetLastError();
}

}  // namespace qm
