/*
 * qm_batch.h -- descriptors of the batch kernel (internal).
 */
#pragma once
#include <stdint.h>

#include "qm_hyp_device.hpp"
#include "qm_internal.h"
#include "qm_student_device.hpp"

namespace qm {

/* Elements of a request per chunk (a workgroup takes one chunk at a time; a
   request's chunks share its tiles in turn): a batch is cut into several
   chunks for each workgroup that the GPU holds at once (batch_chunk), between
   these bounds, in multiples of QM_CHUNK_MIN. */
constexpr uint64_t QM_CHUNK_MIN = 2048;
constexpr uint64_t QM_CHUNK_MAX = 16384;

/* Dynamic LDS (the largest Student t or hyperbolic table of the batch) the batch kernel
   may ask for: 64 KB less its static 8 KB gather list. */
constexpr size_t QM_BATCH_DYNAMIC_LDS_MAX = 65536 - 8192 - 256;

enum BatchOp : uint32_t {
    BOP_NQ64_PLAIN = 0, BOP_NQ64_PAPER, BOP_NQ32_REFINE, BOP_NQ32_PAPER, BOP_NQ32_PLAIN,
    BOP_E64_PLAIN, BOP_E64_PAPER, BOP_E32_REFINE, BOP_T64, BOP_T32, BOP_H64, BOP_H32, BOP_E32_PLAIN,
};

/* Device block: header, then nreq BatchReq. */
struct BatchHeader {
    uint64_t total_chunks;
    uint32_t nreq;
    uint32_t reserved;
    /* per-request completion (the serving loop), or both NULL: for a
       request with `flagged` chunks, count[i] in device memory, 0 at launch,
       counts its finished ones; the workgroup finishing the last sets the
       count back to 0 and the host-visible word done[i], 0 at launch, to 1,
       once every store of the request has reached memory */
    uint32_t* count;
    uint32_t* done;
};

struct BatchReq {
    uint32_t op;            /* BatchOp */
    uint32_t flagged;       /* per-request completion: the request's chunks (0: its batch completes it) */
    const void* in;
    void* out;
    uint64_t n;
    uint64_t chunk_base;    /* global index of the request's first chunk */
    union {
        StudentParams P;    /* Student t: table parameters (cells of the request's dtype) */
        HypParams H;        /* exp -> hyperbolic: table parameters (cells of the request's dtype) */
    };
};

/* A batch of at most BATCH_ARGS_MAX requests, and of no more chunks than the
   launch has workgroups, travels in the kernel's arguments (4 KB at most):
   no upload ordered before the launch. */
constexpr uint32_t BATCH_ARGS_MAX = 16;
struct BatchArgs {
    BatchHeader h;
    BatchReq r[BATCH_ARGS_MAX];
};
static_assert(sizeof(BatchArgs) <= 4096, "kernel arguments");
static_assert(sizeof(BatchHeader) % 8 == 0 && sizeof(BatchReq) % 8 == 0, "uploaded in 8-byte words");

/* The allocation-free entry point's device array: one header and
   QM_BATCH_NOALLOC_MAX_REQUESTS records (736 KiB) per GPU. */
constexpr size_t BATCH_SCRATCH_BYTES = sizeof(BatchHeader) + QM_BATCH_NOALLOC_MAX_REQUESTS * sizeof(BatchReq);
constexpr int BATCH_SCRATCH_MAX_DEVICES = 64;

/* Device address of that array on `device`, which must be the current
   device; looked up on the first call per device and kept (qm_init calls
   it). */
hipError_t batch_scratch_address(int device, void** out);

StudentParams make_params(const TTableHeader& h, const TCells& c, const double* d_rows);
hipError_t launch_batch(const BatchHeader* d_hdr, const BatchReq* d_reqs, size_t lds_bytes, uint64_t blocks,
                        hipStream_t s);
/* Copy `bytes` (a multiple of 8) of pinned host memory to the device, on s. */
hipError_t launch_upload(const void* host, void* dev, size_t bytes, hipStream_t s);
hipError_t launch_batch_args(const BatchArgs& args, size_t lds_bytes, hipStream_t s);

}  // namespace qm
