/*
 * qm_serve.cpp -- batch launch (qm_run_batch) and the continuous-batching
 * serving loop (qm_submit / qm_poll).
 *
 * Batch: requests are validated, Student t tables fetched (built on first
 * use), descriptors written into a pinned staging buffer, copied to the
 * device on the caller's stream and consumed by one launch
 * (qm_batch.hip).  Staging slots are reused once the event recorded after
 * their launch has completed.
 *
 * Serving: qm_submit only validates and queues.  A scheduler thread keeps
 * up to four batches on the device, one per stream.  Whenever a stream is
 * idle it admits the queued requests in arrival order while the bytes of
 * admitted, unfinished requests stay within the context's HBM budget, and
 * launches them as one batch on that stream.  It retires batches whose
 * completion event has fired.  Requests arriving while all streams are busy
 * accumulate into the next batch rather than queueing behind small ones;
 * requests arriving while others run are admitted as a stream and budget
 * free up, and run concurrently with them.
 */
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <mutex>
#include <thread>
#include <unordered_map>
#include <vector>

#include "qm_batch.h"
#include "qm_context.h"
#include "qm_serve.h"

namespace qm {

/* ------------------------------------------------------------------------ */
/* Batch runner                                                             */
/* ------------------------------------------------------------------------ */

/* Per-request completion costs every chunk of a flagged request an L2
   write-back and a count, 64 ns each beside the streams and one after the
   other (MI355X: 1100 flagged chunks took 80 us where the batch's work takes
   14).  So only requests of at most sixteen chunks are flagged, and as many
   of a batch's, in order, as cost it a third of its time at about 350 G
   elements/s: one chunk for each 2^16 elements.  That covers the small
   requests beside large ones, which gain by it (median until a request is
   observed complete: 200 of 2^15 elements before one of 2^26 117 us, 240 with
   one chunk for each 2^20 elements, 100 of 2^17 before 2^26 138 and 255; 8 of
   2^12 in a batch of under 2^24 22, 82 with such batches unflagged), and
   leaves a batch of nothing but small ones mostly to its event, which is then
   the earlier of the two (512 of 2^15: 90 us, 445 with every request flagged).
   2000 requests of 2^12..2^24 elements at once run at 330 G elements/s with
   this, 345 with the smaller budget.  A batch of under 2^22 elements is over
   within some 20 us and has no flags (8 requests of 2^10..2^18: 42 us, 47 with
   them). */
constexpr uint64_t FLAG_MIN_ELEMENTS = 1 << 22, FLAG_ELEMENTS_PER_CHUNK = 1 << 16;
static uint64_t batch_flag_chunks()
{
    /* tuning: QM_SERVE_FLAG_CHUNKS overrides the limit (0: completion by
       batch only) */
    static const uint64_t v = [] {
        const char* e = getenv("QM_SERVE_FLAG_CHUNKS");
        return e ? (uint64_t)strtoull(e, nullptr, 10) : (uint64_t)16;
    }();
    return v;
}

/* Requests per batch that get a completion flag (a batch with more relies
   on its event alone); one host-coherent array of this many words and one of
   chunk counts in device memory per serving stream. */
constexpr size_t SERVE_FLAGS = 4096;

struct Staging {
    void* host = nullptr;
    void* dev = nullptr;
    size_t cap = 0;
    hipEvent_t ev = nullptr;
    bool busy = false;         /* held by a caller between acquire and event record */
};

struct BatchRunner {
    std::mutex mu;
    std::vector<Staging*> slots;
    size_t next = 0;           /* ring position: the oldest use is tried first */
};

static BatchRunner* runner_of(qm_ctx* ctx)
{
    std::lock_guard<std::mutex> lk(ctx->server_mu);
    if (!ctx->runner) ctx->runner = new BatchRunner;
    return ctx->runner;
}

void runner_free(qm_ctx* ctx)
{
    BatchRunner* r = ctx->runner;
    if (!r) return;
    for (Staging* s : r->slots) {
        if (s->ev) {
            (void)hipEventSynchronize(s->ev);
            (void)hipEventDestroy(s->ev);
        }
        if (s->host) (void)hipHostFree(s->host);
        if (s->dev) (void)hipFree(s->dev);
        delete s;
    }
    delete r;
    ctx->runner = nullptr;
}

static Staging* new_slot()
{
    Staging* s = new Staging;
    if (hipEventCreateWithFlags(&s->ev, hipEventDisableTiming) == hipSuccess) return s;
    delete s;
    return nullptr;
}

/* At least `bytes` of pinned host and device memory in a slot not in use. */
static bool size_slot(Staging* s, size_t bytes)
{
    if (s->cap >= bytes) return true;
    if (s->host) (void)hipHostFree(s->host);
    if (s->dev) (void)hipFree(s->dev);
    s->host = s->dev = nullptr;
    s->cap = 0;
    const size_t cap = std::max(bytes, (size_t)1 << 16);
    if (hipHostMalloc(&s->host, cap, hipHostMallocDefault) != hipSuccess || hipMalloc(&s->dev, cap) != hipSuccess)
        return false;
    s->cap = cap;
    return true;
}

/* A staging slot with at least `bytes` of pinned host and device memory,
   whose previous use has completed. */
static qm_status acquire_slot(BatchRunner* br, size_t bytes, Staging** out)
{
    std::unique_lock<std::mutex> lk(br->mu);
    Staging* slot = nullptr;
    /* slots are used in ring order, so the one at `next` holds the oldest
       launch: one event query usually settles it; otherwise add a slot */
    const size_t ns = br->slots.size();
    for (size_t k = 0; k < ns && k < 2 && !slot; ++k) {
        Staging* s = br->slots[(br->next + k) % ns];
        if (!s->busy && hipEventQuery(s->ev) == hipSuccess) {
            slot = s;
            br->next = (br->next + k + 1) % ns;
        }
    }
    if (!slot && ns < 32) {
        slot = new_slot();
        if (!slot) return set_error(QM_E_HIP, "hipEventCreate failed");
        br->slots.insert(br->slots.begin() + br->next, slot);
        br->next = (br->next + 1) % br->slots.size();
    }
    while (!slot) {             /* all 32 in use: take the oldest that no caller holds */
        for (size_t k = 0; k < br->slots.size() && !slot; ++k) {
            Staging* s = br->slots[(br->next + k) % br->slots.size()];
            if (!s->busy) {
                slot = s;
                br->next = (br->next + k + 1) % br->slots.size();
            }
        }
        if (!slot) {
            lk.unlock();
            std::this_thread::yield();
            lk.lock();
        }
    }
    slot->busy = true;
    lk.unlock();
    (void)hipEventSynchronize(slot->ev);
    if (!size_slot(slot, bytes)) {
        std::lock_guard<std::mutex> g(br->mu);
        slot->busy = false;
        return set_error(QM_E_NOMEM, "staging allocation failed");
    }
    *out = slot;
    return QM_OK;
}

static uint32_t batch_op(const qm_request& r)
{
    switch (r.kind) {
    case QM_NORMAL_QUANTILE:
        if (r.dtype == QM_F64) return r.mode == QM_PAPER ? BOP_NQ64_PAPER : BOP_NQ64_PLAIN;
        if (r.mode == QM_F32_REFINE) return BOP_NQ32_REFINE;
        return r.mode == QM_PAPER ? BOP_NQ32_PAPER : BOP_NQ32_PLAIN;
    case QM_EXP_TO_NORMAL:
        if (r.dtype == QM_F64) return r.mode == QM_PAPER ? BOP_E64_PAPER : BOP_E64_PLAIN;
        return r.mode == QM_PLAIN ? BOP_E32_PLAIN : BOP_E32_REFINE;
    case QM_EXP_TO_HYPERBOLIC:
    case QM_EXP_TO_VG:
        return r.dtype == QM_F64 ? BOP_H64 : BOP_H32;
    default:
        return r.dtype == QM_F64 ? BOP_T64 : BOP_T32;
    }
}

/* Chunk size of a batch of total_n elements: about BATCH_ROUNDS chunks for
   each of the cus x 4 workgroups that the GPU holds at once, within
   [chunk_floor, QM_CHUNK_MAX], a multiple of QM_CHUNK_MIN.  Fewer, larger
   chunks leave the last of them running alone, more pay the start of a
   chunk (descriptor, table, first loads) too often: 512 requests of
   2^10..2^20 elements take 177 us a pass with 4 rounds, 166 with 8, 172 with
   12; 4096 requests of 2^10..2^22 elements 4.97 ms in chunks of 16384, 5.30 of
   32768, 5.06 of 8192.  A lone request is spread over the whole GPU: of 2^15 elements it took
   30 us in one chunk of that size, and takes 6 in sixteen. */
constexpr uint64_t BATCH_ROUNDS = 8;
static uint64_t batch_chunk(uint64_t total_n, int cus)
{
    static const uint64_t chunk_floor = [] {
        /* tuning: lower bound of the chunk size */
        const char* e = getenv("QM_BATCH_CHUNK_MIN");
        uint64_t v = e ? strtoull(e, nullptr, 10) : QM_CHUNK_MIN;
        v = (v / QM_CHUNK_MIN) * QM_CHUNK_MIN;
        return v < QM_CHUNK_MIN ? QM_CHUNK_MIN : (v > QM_CHUNK_MAX ? QM_CHUNK_MAX : v);
    }();
    uint64_t chunk = total_n / ((uint64_t)cus * 4 * BATCH_ROUNDS);
    chunk = (chunk / QM_CHUNK_MIN) * QM_CHUNK_MIN;
    return chunk < chunk_floor ? chunk_floor : (chunk > QM_CHUNK_MAX ? QM_CHUNK_MAX : chunk);
}

static uint64_t batch_blocks(const qm_ctx* ctx, uint64_t chunks)
{
    /* a workgroup per chunk up to 1024 per compute unit: the hardware hands
       the next one to whichever unit is free, which evens out chunks of
       different kinds (512 requests of 2^10..2^20 elements: 186 us a pass,
       198 with 8 per unit; 4096 of 2^10..2^22: 5.13 ms, 5.28 with 64) */
    uint64_t blocks = (uint64_t)ctx->cus * 1024;
    return blocks > chunks ? chunks : blocks;
}

/*
 * The descriptors of a validated batch, in request order (requests with
 * n = 0 are skipped), each handed to emit(const BatchReq&); h receives the
 * header.  Tables the requests need are fetched from the context and, when
 * build_tables, built on first use; otherwise a missing table is an error.
 */
template <class Emit>
static qm_status plan_batch(qm_ctx* ctx, const qm_request* reqs, uint64_t count, bool build_tables, BatchHeader* h,
                            size_t* lds_out, Emit emit)
{
    uint64_t total_n = 0;
    for (uint64_t i = 0; i < count; ++i) total_n += reqs[i].n;
    const uint64_t chunk = batch_chunk(total_n, ctx->cus);
    uint64_t chunks = 0;
    uint32_t nreq = 0;
    size_t lds = 0;
    for (uint64_t i = 0; i < count; ++i) {
        const qm_request& r = reqs[i];
        if (r.n == 0) continue;
        BatchReq b;
        memset(&b, 0, sizeof b);
        b.op = batch_op(r);
        b.in = r.d_in;
        b.out = r.d_out;
        b.n = r.n;
        b.chunk_base = chunks;
        chunks += (r.n + chunk - 1) / chunk;
        if (r.kind == QM_STUDENT_T) {
            const DeviceTable* t = nullptr;
            qm_status st = build_tables ? get_table(ctx, r.nu, &t) : find_table(ctx, r.nu, &t);
            if (st != QM_OK) return st;
            const TCells& c = r.dtype == QM_F64 ? t->hdr.f64 : t->hdr.f32;
            b.P = make_params(t->hdr, c, table_block(t->d_table) + c.coef_offset);
            if (!t->hdr.identity) lds = std::max(lds, student_lds_bytes(b.P));
        } else if (r.kind == QM_EXP_TO_HYPERBOLIC || r.kind == QM_EXP_TO_VG) {
            const bool vg = r.kind == QM_EXP_TO_VG;
            const DeviceHypTable* t = nullptr;
            qm_status st = vg ? (build_tables ? get_vg_table(ctx, r.nu, r.alpha, r.beta, &t)
                                              : find_base_table(ctx, true, r.nu, r.alpha, r.beta, &t))
                              : (build_tables ? get_hyp_table(ctx, r.alpha, r.beta, r.delta, &t)
                                              : find_base_table(ctx, false, r.alpha, r.beta, r.delta, &t));
            if (st != QM_OK) return st;
            size_t l = 0;
            if (!make_hyp_params(t->hdr, r.dtype == QM_F32, t->d_table, t->ncoef, r.mu, &b.H, &l))
                return set_error(QM_E_INVAL, "invalid hyperbolic table");
            lds = std::max(lds, l);
        }
        qm_status st = emit(b);
        if (st != QM_OK) return st;
        ++nreq;
    }
    if (lds > QM_BATCH_DYNAMIC_LDS_MAX) return set_error(QM_E_INVAL, "table larger than the LDS a launch may use");
    memset(h, 0, sizeof *h);
    h->total_chunks = chunks;
    h->nreq = nreq;
    *lds_out = lds;
    return QM_OK;
}

static qm_status validate_batch(qm_ctx* ctx, const qm_request* reqs, uint64_t count)
{
    if (!ctx) return set_error(QM_E_INVAL, "context is NULL");
    if (count > 0 && !reqs) return set_error(QM_E_INVAL, "reqs is NULL");
    for (uint64_t i = 0; i < count; ++i) {
        qm_status st = check_request(reqs[i], nullptr, false);
        if (st != QM_OK) return st;
    }
    if (hipSetDevice(ctx->device) != hipSuccess) return set_error(QM_E_HIP, "hipSetDevice failed");
    return QM_OK;
}

/* Whether a planned batch travels in the kernel's arguments. */
static bool fits_args(const qm_ctx* ctx, const BatchHeader& h)
{
    return h.nreq <= BATCH_ARGS_MAX && h.total_chunks <= (uint64_t)ctx->cus * 8;
}

static hipError_t launch_in_args(const BatchHeader& h, const BatchReq* reqs, size_t lds, hipStream_t s)
{
    BatchArgs a;
    a.h = h;
    memcpy(a.r, reqs, h.nreq * sizeof(BatchReq));
    return launch_batch_args(a, lds, s);
}

/*
 * Validate and enqueue `count` requests as one launch on s.  If
 * done is not NULL, an event that completes with the launch is recorded
 * into it (the caller owns the event).
 */
qm_status enqueue_batch(qm_ctx* ctx, const qm_request* reqs, uint64_t count, hipStream_t s, hipEvent_t done,
                        uint32_t* flags, uint32_t* counts)
{
    qm_status st = validate_batch(ctx, reqs, count);
    if (st != QM_OK) return st;
    std::vector<BatchReq> d;
    d.reserve(count);
    BatchHeader h;
    size_t lds = 0;
    st = plan_batch(ctx, reqs, count, true, &h, &lds, [&](const BatchReq& b) {
        d.push_back(b);
        return (qm_status)QM_OK;
    });
    if (st != QM_OK) return st;
    if (d.empty()) {
        if (done && hipEventRecord(done, s) != hipSuccess) return set_error(QM_E_HIP, "hipEventRecord failed");
        return QM_OK;
    }
    if (fits_args(ctx, h)) {        /* over within some 20 us: its event completes it */
        hipError_t e = launch_in_args(h, d.data(), lds, s);
        if (e != hipSuccess) return set_error(QM_E_HIP, hipGetErrorString(e));
        if (done && hipEventRecord(done, s) != hipSuccess) return set_error(QM_E_HIP, "hipEventRecord failed");
        return QM_OK;
    }
    if (flags) {
        uint64_t total = 0, budget = 0;
        for (const BatchReq& r : d) total += r.n;
        budget = total < FLAG_MIN_ELEMENTS ? 0 : total / FLAG_ELEMENTS_PER_CHUNK;
        for (size_t i = 0; i < d.size(); ++i) {
            BatchReq& r = d[i];
            const uint64_t c = (i + 1 < d.size() ? d[i + 1].chunk_base : h.total_chunks) - r.chunk_base;
            if (c > batch_flag_chunks() || c > budget) continue;
            budget -= c;
            r.flagged = (uint32_t)c;
            h.count = counts;
            h.done = flags;
        }
    }
    const size_t bytes = sizeof(BatchHeader) + d.size() * sizeof(BatchReq);
    Staging* slot = nullptr;
    st = acquire_slot(runner_of(ctx), bytes, &slot);
    if (st != QM_OK) return st;
    memcpy(slot->host, &h, sizeof h);
    memcpy((char*)slot->host + sizeof h, d.data(), d.size() * sizeof(BatchReq));
    hipError_t e = launch_upload(slot->host, slot->dev, bytes, s);
    if (e == hipSuccess)
        e = launch_batch((const BatchHeader*)slot->dev, (const BatchReq*)((char*)slot->dev + sizeof h), lds,
                         batch_blocks(ctx, h.total_chunks), s);
    hipError_t e2 = hipEventRecord(slot->ev, s);
    {
        std::lock_guard<std::mutex> g(runner_of(ctx)->mu);
        slot->busy = false;
    }
    if (e != hipSuccess) return set_error(QM_E_HIP, hipGetErrorString(e));
    if (e2 != hipSuccess) return set_error(QM_E_HIP, hipGetErrorString(e2));
    if (done && hipEventRecord(done, s) != hipSuccess) return set_error(QM_E_HIP, "hipEventRecord failed");
    return QM_OK;
}

/*
 * The allocation-free form of enqueue_batch: descriptors are planned into
 * the context's pinned host buffer (once the previous upload from it has
 * completed), copied to the GPU's fixed descriptor array on s and launched
 * from there.  No table is built and nothing is allocated.
 */
qm_status enqueue_batch_noalloc(qm_ctx* ctx, const qm_request* reqs, uint64_t count, hipStream_t s)
{
    qm_status st = validate_batch(ctx, reqs, count);
    if (st != QM_OK) return st;
    uint64_t live = 0;
    for (uint64_t i = 0; i < count; ++i) live += reqs[i].n != 0;
    if (live > QM_BATCH_NOALLOC_MAX_REQUESTS) {
        char msg[160];
        snprintf(msg, sizeof msg, "%llu requests with n > 0; the allocation-free batch takes at most %d",
                 (unsigned long long)live, QM_BATCH_NOALLOC_MAX_REQUESTS);
        return set_error(QM_E_INVAL, msg);
    }
    if (!ctx->noalloc_dev || !ctx->noalloc_host || !ctx->noalloc_ev)
        return set_error(QM_E_HIP, "allocation-free batch path not set up");
    std::lock_guard<std::mutex> lk(ctx->noalloc_mu);
    hipError_t e = hipEventSynchronize(ctx->noalloc_ev);
    if (e != hipSuccess) return set_error(QM_E_HIP, hipGetErrorString(e));
    BatchHeader h;
    size_t lds = 0;
    BatchReq* staged = reinterpret_cast<BatchReq*>(static_cast<char*>(ctx->noalloc_host) + sizeof(BatchHeader));
    uint64_t k = 0;
    st = plan_batch(ctx, reqs, count, false, &h, &lds, [&](const BatchReq& b) {
        staged[k++] = b;
        return (qm_status)QM_OK;
    });
    if (st != QM_OK) return st;
    if (k == 0) return QM_OK;
    if (fits_args(ctx, h)) {
        e = launch_in_args(h, staged, lds, s);
        if (e != hipSuccess) return set_error(QM_E_HIP, hipGetErrorString(e));
        return QM_OK;
    }
    memcpy(ctx->noalloc_host, &h, sizeof h);
    const size_t bytes = sizeof(BatchHeader) + k * sizeof(BatchReq);
    e = launch_upload(ctx->noalloc_host, ctx->noalloc_dev, bytes, s);
    if (e == hipSuccess) e = hipEventRecord(ctx->noalloc_ev, s);
    if (e == hipSuccess)
        e = launch_batch(static_cast<const BatchHeader*>(ctx->noalloc_dev),
                         reinterpret_cast<const BatchReq*>(static_cast<char*>(ctx->noalloc_dev) + sizeof h), lds,
                         batch_blocks(ctx, h.total_chunks), s);
    if (e != hipSuccess) return set_error(QM_E_HIP, hipGetErrorString(e));
    return QM_OK;
}

/* ------------------------------------------------------------------------ */
/* Serving loop                                                             */
/* ------------------------------------------------------------------------ */

typedef std::chrono::steady_clock clk;

enum TicketState { T_QUEUED = 0, T_RUNNING = 1, T_DONE = 2, T_CLOSED = 3, T_FAILED = 4 };

struct Ticket {
    qm_request req;
    uint64_t bytes;
    int state;
    clk::time_point t_submit;
    clk::time_point t_done;
};

/* Finished tickets are kept for the most recent SERVE_KEEP_FINISHED
   completions (then forgotten: qm_poll reports QM_E_TICKET); latencies for
   the most recent SERVE_KEEP_LATENCIES.  Both bound a long-running
   server's memory. */
constexpr size_t SERVE_KEEP_FINISHED = 1 << 16;
constexpr size_t SERVE_KEEP_LATENCIES = 1 << 20;

struct InFlight {
    hipEvent_t ev;
    std::vector<uint64_t> tickets;
    uint64_t bytes;             /* of the tickets not yet observed complete */
    int stream;
    /* per-request completion: flag[k] is ticket k's word in its stream's
       flag array, or -1 (n = 0, or no flags: the batch's event completes it) */
    std::vector<int32_t> flag;
    uint32_t* flags;
    bool ended;                 /* its event has fired */
};

constexpr int SERVE_STREAMS = 4;
/* How long the scheduler stays awake after its last batch. */
constexpr std::chrono::microseconds SERVE_IDLE_SPIN(50);

struct Server {
    qm_ctx* ctx = nullptr;
    std::thread th;
    /* mu guards the queue, the tickets and the counters: what submitters,
       pollers and the scheduler share, each for a few hundred nanoseconds.
       Streams, batches in flight and events are the scheduler's own, so that
       its device queries hold up nobody. */
    std::mutex mu;
    std::condition_variable cv;
    std::deque<uint64_t> queue;
    std::atomic<uint64_t> queued{0};      /* queue.size(), readable without mu */
    std::atomic<bool> stop{false};        /* set under mu */
    bool waiting = false;                 /* the scheduler sleeps on cv */
    std::unordered_map<uint64_t, Ticket> tickets;
    uint64_t next_ticket = 1;
    uint64_t in_flight_bytes = 0;
    std::deque<uint64_t> finished;        /* terminal tickets, oldest first */
    std::vector<uint64_t> latencies_ns;   /* ring of SERVE_KEEP_LATENCIES */
    uint64_t completed = 0, failed = 0, submitted = 0;
    uint64_t in_flight_bytes_hwm = 0;
    uint64_t in_flight_requests = 0;
    hipStream_t streams[SERVE_STREAMS] = {};
    bool stream_busy[SERVE_STREAMS] = {};
    uint32_t* flags[SERVE_STREAMS] = {};  /* host-coherent, device-visible; NULL: events only */
    uint32_t* counts[SERVE_STREAMS] = {}; /* chunk counts beside them, all 0 between launches */
    std::vector<InFlight> inflight;
    std::vector<hipEvent_t> free_events;
};

/* A ticket reached a terminal state: keep it among the recent ones. */
static void finish_ticket(Server* S, uint64_t t)
{
    S->finished.push_back(t);
    while (S->finished.size() > SERVE_KEEP_FINISHED) {
        S->tickets.erase(S->finished.front());
        S->finished.pop_front();
    }
}

/* Ticket k of in-flight batch f observed complete at `now`. */
static void complete_ticket(Server* S, InFlight& f, size_t k, clk::time_point now)
{
    const uint64_t t = f.tickets[k];
    auto it = S->tickets.find(t);
    /* already complete by its flag (and perhaps forgotten since) */
    if (it == S->tickets.end() || it->second.state == T_DONE) return;
    Ticket& tk = it->second;
    tk.state = T_DONE;
    tk.t_done = now;
    uint64_t lat = (uint64_t)std::chrono::duration_cast<std::chrono::nanoseconds>(now - tk.t_submit).count();
    if (S->latencies_ns.size() < SERVE_KEEP_LATENCIES) S->latencies_ns.push_back(lat);
    else S->latencies_ns[S->completed % SERVE_KEEP_LATENCIES] = lat;
    ++S->completed;
    --S->in_flight_requests;
    S->in_flight_bytes -= tk.bytes;
    f.bytes -= tk.bytes;
    finish_ticket(S, t);
}

static void server_loop(Server* S)
{
    (void)hipSetDevice(S->ctx->device);
    /* completion polling while batches are on the device: spin with yields
       (default; measured: p50 0.08 ms against 0.09-0.11 ms with a 20 us timed
       wait, p99 at 50k req/s 1.6 ms against 1.8 ms), or a timed wait of
       QM_SERVE_POLL_US microseconds (tuning) */
    static const long poll_us = [] {
        const char* e = getenv("QM_SERVE_POLL_US");
        long v = e ? strtol(e, nullptr, 10) : 0;
        return v < 0 ? 0 : v;
    }();
    std::vector<uint64_t> admit;
    std::vector<qm_request> reqs;
    std::vector<std::pair<size_t, size_t>> seen;   /* (batch, ticket of it) observed complete */
    clk::time_point last_work = clk::now();
    for (;;) {
        /* complete requests whose flag is up, and retire finished batches
           (their event completes whatever the flags have not) */
        seen.clear();
        bool ended = false;
        for (size_t i = 0; i < S->inflight.size(); ++i) {
            InFlight& f = S->inflight[i];
            f.ended = hipEventQuery(f.ev) == hipSuccess;
            ended |= f.ended;
            if (!f.ended && !f.flags) continue;
            for (size_t k = 0; k < f.tickets.size(); ++k)
                if (f.ended || (f.flag[k] >= 0 && __atomic_load_n(f.flags + f.flag[k], __ATOMIC_ACQUIRE) != 0)) {
                    seen.emplace_back(i, k);
                    f.flag[k] = -1;
                }
        }
        if (!seen.empty()) {
            std::lock_guard<std::mutex> lk(S->mu);
            const clk::time_point now = clk::now();
            for (const auto& c : seen) complete_ticket(S, S->inflight[c.first], c.second, now);
        }
        for (size_t i = 0; ended && i < S->inflight.size();) {
            InFlight& f = S->inflight[i];
            if (f.ended) {
                S->stream_busy[f.stream] = false;
                S->free_events.push_back(f.ev);
                S->inflight.erase(S->inflight.begin() + i);
            } else {
                ++i;
            }
        }
        /* continuous batching: a batch is formed only when a stream is idle,
           from everything queued by then (in arrival order, within the
           budget); while all streams are busy, arrivals accumulate into the
           next, larger batch rather than queueing behind small ones */
        admit.clear();
        reqs.clear();
        uint64_t bytes = 0;
        int idle = -1;
        for (int k = 0; k < SERVE_STREAMS; ++k)
            if (!S->stream_busy[k]) { idle = k; break; }
        const bool stop = S->stop;
        if (!stop && idle >= 0 && S->queued > 0) {
            std::lock_guard<std::mutex> lk(S->mu);
            while (!S->queue.empty()) {
                Ticket& tk = S->tickets[S->queue.front()];
                if (S->in_flight_bytes + bytes + tk.bytes > S->ctx->budget) break;
                bytes += tk.bytes;
                tk.state = T_RUNNING;
                admit.push_back(S->queue.front());
                reqs.push_back(tk.req);
                S->queue.pop_front();
                --S->queued;
            }
            S->in_flight_bytes += bytes;
            S->in_flight_requests += admit.size();
            if (S->in_flight_bytes > S->in_flight_bytes_hwm) S->in_flight_bytes_hwm = S->in_flight_bytes;
        }
        if (admit.empty()) {
            const clk::time_point now = clk::now();
            if (!S->inflight.empty()) last_work = now;
            if (S->inflight.empty() && (stop || now - last_work > SERVE_IDLE_SPIN)) {
                std::unique_lock<std::mutex> lk(S->mu);
                if (S->stop) {
                    for (uint64_t t : S->queue) {
                        S->tickets[t].state = T_CLOSED;
                        finish_ticket(S, t);
                    }
                    S->queue.clear();
                    S->queued = 0;
                    return;
                }
                S->waiting = true;
                S->cv.wait(lk, [S] { return S->stop || !S->queue.empty(); });
                S->waiting = false;
                last_work = clk::now();
            } else if (poll_us == 0 || S->inflight.empty()) {
                /* work on the device: poll again at once (a timed wait
                   oversleeps by tens of microseconds, which every request
                   would pay), as for a moment after the last of it (a
                   sleeping scheduler costs the next submitter a wake-up) */
                std::this_thread::yield();
            } else {
                std::unique_lock<std::mutex> lk(S->mu);
                S->waiting = true;
                S->cv.wait_for(lk, std::chrono::microseconds(poll_us));
                S->waiting = false;
            }
            continue;
        }
        /* completion flags: one word per request with n > 0, in order */
        std::vector<int32_t> flag(admit.size(), -1);
        uint32_t* flags = S->flags[idle];
        int32_t live = 0;
        for (size_t k = 0; k < reqs.size(); ++k)
            if (reqs[k].n > 0) flag[k] = live++;
        if (flags && (size_t)live <= SERVE_FLAGS) {
            for (int32_t k = 0; k < live; ++k) __atomic_store_n(flags + k, 0u, __ATOMIC_RELAXED);
        } else {
            flags = nullptr;
            std::fill(flag.begin(), flag.end(), -1);
        }
        hipEvent_t ev = nullptr;
        if (!S->free_events.empty()) { ev = S->free_events.back(); S->free_events.pop_back(); }
        hipStream_t st = S->streams[idle];
        S->stream_busy[idle] = true;
        if (!ev) (void)hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        qm_status rc = enqueue_batch(S->ctx, reqs.data(), reqs.size(), st, ev, flags, S->counts[idle]);
        if (rc != QM_OK) {
            std::lock_guard<std::mutex> lk(S->mu);
            for (uint64_t t : admit) {
                S->tickets[t].state = T_FAILED;
                finish_ticket(S, t);
            }
            S->failed += admit.size();
            S->in_flight_requests -= admit.size();
            S->in_flight_bytes -= bytes;
            S->stream_busy[idle] = false;
            S->free_events.push_back(ev);
            continue;
        }
        S->inflight.push_back(InFlight{ev, admit, bytes, idle, std::move(flag), flags, false});
    }
}

/*
 * Completion flags of serving stream i, in pinned host memory that the GPU
 * writes through to while a batch runs, and the chunk counts beside them.  A
 * stream carries one batch at a time and every launch leaves the counts 0, so
 * they are cleared here once, by a copy kernel on that stream: the scheduler
 * allocates nothing for them, and nothing waits for the caller's own streams
 * (a synchronous copy is ordered after all work on the default one).
 * Without them (an allocation failed) every request completes with its
 * batch's event.
 */
static void make_flags(Server* S, int i)
{
    const size_t bytes = SERVE_FLAGS * sizeof(uint32_t);
    void *flags = nullptr, *counts = nullptr;
    bool ok = hipHostMalloc(&flags, bytes, hipHostMallocCoherent) == hipSuccess &&
              hipMalloc(&counts, bytes) == hipSuccess;
    if (ok) {
        memset(flags, 0, bytes);
        ok = launch_upload(flags, counts, bytes, S->streams[i]) == hipSuccess;
    }
    if (!ok) {
        if (counts) (void)hipFree(counts);
        if (flags) (void)hipHostFree(flags);
        (void)hipGetLastError();
        return;
    }
    S->flags[i] = static_cast<uint32_t*>(flags);
    S->counts[i] = static_cast<uint32_t*>(counts);
}

static void free_flags(Server* S)
{
    for (int i = 0; i < SERVE_STREAMS; ++i) {
        if (S->flags[i]) (void)hipHostFree(S->flags[i]);
        if (S->counts[i]) (void)hipFree(S->counts[i]);
    }
}

/* Staging slots for the serving loop, made before it starts: a batch on each
   stream and as many that have just ended.  One made for a batch in traffic
   holds up the scheduler for its allocations, and the first 500 requests at
   50k a second had a p99 of 0.38..0.53 ms on MI355X, 0.14..0.19 with the slots
   made here. */
static void reserve_slots(BatchRunner* br)
{
    std::lock_guard<std::mutex> lk(br->mu);
    while (br->slots.size() < 2 * SERVE_STREAMS) {
        Staging* s = new_slot();
        if (!s) return;
        br->slots.push_back(s);
        if (!size_slot(s, 1)) {
            (void)hipGetLastError();
            return;
        }
    }
}

static Server* server_of(qm_ctx* ctx, qm_status* st)
{
    std::lock_guard<std::mutex> lk(ctx->server_mu);
    if (ctx->server) return ctx->server;
    Server* S = new Server;
    S->ctx = ctx;
    (void)hipSetDevice(ctx->device);
    for (int i = 0; i < SERVE_STREAMS; ++i) {
        if (hipStreamCreateWithFlags(&S->streams[i], hipStreamNonBlocking) != hipSuccess) {
            for (int j = 0; j < i; ++j) {
                (void)hipStreamSynchronize(S->streams[j]);
                (void)hipStreamDestroy(S->streams[j]);
            }
            free_flags(S);
            delete S;
            *st = set_error(QM_E_HIP, "hipStreamCreate failed");
            return nullptr;
        }
        make_flags(S, i);
    }
    if (!ctx->runner) ctx->runner = new BatchRunner;
    reserve_slots(ctx->runner);
    S->th = std::thread(server_loop, S);
    ctx->server = S;
    return S;
}

void server_stop(Server* S)
{
    if (!S) return;
    {
        std::lock_guard<std::mutex> lk(S->mu);
        S->stop = true;
    }
    S->cv.notify_all();
    if (S->th.joinable()) S->th.join();
    for (InFlight& f : S->inflight) {
        (void)hipEventSynchronize(f.ev);
        (void)hipEventDestroy(f.ev);
    }
    for (hipEvent_t e : S->free_events) (void)hipEventDestroy(e);
    for (int i = 0; i < SERVE_STREAMS; ++i)
        if (S->streams[i]) {
            (void)hipStreamSynchronize(S->streams[i]);
            (void)hipStreamDestroy(S->streams[i]);
        }
    free_flags(S);
    delete S;
}

}  // namespace qm

extern "C" {

qm_status qm_run_batch(qm_ctx* ctx, const qm_request* reqs, uint64_t count, void* hip_stream)
{
    return qm::enqueue_batch(ctx, reqs, count, (hipStream_t)hip_stream, nullptr);
}

qm_status qm_run_batch_noalloc(qm_ctx* ctx, const qm_request* reqs, uint64_t count, void* hip_stream)
{
    return qm::enqueue_batch_noalloc(ctx, reqs, count, (hipStream_t)hip_stream);
}

qm_status qm_submit(qm_ctx* ctx, const qm_request* req, uint64_t* ticket)
{
    if (!ctx || !req || !ticket) return qm::set_error(QM_E_INVAL, "NULL argument");
    int es = 0;
    qm_status st = qm::check_request(*req, &es, false);
    if (st != QM_OK) return st;
    uint64_t bytes = 2 * req->n * (uint64_t)es;
    if (bytes > ctx->budget) return qm::set_error(QM_E_INVAL, "request larger than the HBM budget");
    /* a table the request needs is built here, in the caller's thread, so
       that the scheduler never stalls on a build and a failed build is this
       request's error alone */
    if (req->kind == QM_STUDENT_T || req->kind == QM_EXP_TO_HYPERBOLIC || req->kind == QM_EXP_TO_VG) {
        if (hipSetDevice(ctx->device) != hipSuccess) return qm::set_error(QM_E_HIP, "hipSetDevice failed");
        if (req->kind == QM_STUDENT_T) {
            const DeviceTable* t = nullptr;
            st = qm::get_table(ctx, req->nu, &t);
        } else if (req->kind == QM_EXP_TO_VG) {
            const DeviceHypTable* t = nullptr;
            st = qm::get_vg_table(ctx, req->nu, req->alpha, req->beta, &t);
        } else {
            const DeviceHypTable* t = nullptr;
            st = qm::get_hyp_table(ctx, req->alpha, req->beta, req->delta, &t);
        }
        if (st != QM_OK) return st;
    }
    st = QM_OK;
    qm::Server* S = qm::server_of(ctx, &st);
    if (!S) return st;
    bool wake;
    {
        std::lock_guard<std::mutex> lk(S->mu);
        if (S->stop) return qm::set_error(QM_E_CLOSED, "serving loop is shutting down");
        uint64_t t = S->next_ticket++;
        qm::Ticket tk;
        tk.req = *req;
        tk.bytes = bytes;
        tk.state = qm::T_QUEUED;
        tk.t_submit = qm::clk::now();
        S->tickets.emplace(t, tk);
        S->queue.push_back(t);
        ++S->queued;
        ++S->submitted;
        *ticket = t;
        wake = S->waiting;
    }
    if (wake) S->cv.notify_one();
    return QM_OK;
}

static qm::Server* server_if_any(qm_ctx* ctx)
{
    std::lock_guard<std::mutex> lk(ctx->server_mu);
    return ctx->server;
}

static uint64_t steady_ns(qm::clk::time_point t)
{
    return (uint64_t)std::chrono::duration_cast<std::chrono::nanoseconds>(t.time_since_epoch()).count();
}

qm_status qm_poll_times(qm_ctx* ctx, uint64_t ticket, uint64_t* submit_ns, uint64_t* done_ns)
{
    if (!ctx) return qm::set_error(QM_E_INVAL, "context is NULL");
    qm::Server* S = server_if_any(ctx);
    if (!S) return qm::set_error(QM_E_TICKET, "unknown ticket");
    std::lock_guard<std::mutex> lk(S->mu);
    auto it = S->tickets.find(ticket);
    if (it == S->tickets.end()) return qm::set_error(QM_E_TICKET, "unknown or forgotten ticket");
    if (submit_ns) *submit_ns = steady_ns(it->second.t_submit);
    switch (it->second.state) {
    case qm::T_DONE:
        if (done_ns) *done_ns = steady_ns(it->second.t_done);
        return QM_OK;
    case qm::T_CLOSED: return qm::set_error(QM_E_CLOSED, "request failed by shutdown");
    case qm::T_FAILED: return qm::set_error(QM_E_HIP, "request launch failed");
    default: return QM_PENDING;
    }
}

qm_status qm_poll(qm_ctx* ctx, uint64_t ticket) { return qm_poll_times(ctx, ticket, nullptr, nullptr); }

uint64_t qm_serving_latencies(qm_ctx* ctx, uint64_t* lat_ns, uint64_t cap)
{
    if (!ctx) return 0;
    qm::Server* S = server_if_any(ctx);
    if (!S) return 0;
    std::lock_guard<std::mutex> lk(S->mu);
    const uint64_t kept = S->latencies_ns.size();
    if (lat_ns && kept) {
        /* the most recent min(cap, kept), oldest first; once the ring has
           wrapped, its oldest entry is at completed mod its size */
        uint64_t m = cap < kept ? cap : kept;
        uint64_t start = (S->completed - m) % qm::SERVE_KEEP_LATENCIES;
        for (uint64_t i = 0; i < m; ++i) {
            uint64_t j = kept < qm::SERVE_KEEP_LATENCIES ? (S->completed - m + i) : (start + i) % kept;
            lat_ns[i] = S->latencies_ns[j];
        }
    }
    return S->completed;
}

/* Staging slots made so far (include/qm_debug.h). */
int qm_debug_staging_slots(void* ctx)
{
    qm::BatchRunner* br = ctx ? qm::runner_of(static_cast<qm_ctx*>(ctx)) : nullptr;
    if (!br) return -1;
    std::lock_guard<std::mutex> lk(br->mu);
    return (int)br->slots.size();
}

qm_status qm_serving_stats(qm_ctx* ctx, qm_serving_counters* out)
{
    if (!ctx || !out) return qm::set_error(QM_E_INVAL, "NULL argument");
    memset(out, 0, sizeof *out);
    out->budget_bytes = ctx->budget;
    qm::Server* S = server_if_any(ctx);
    if (!S) return QM_OK;
    std::lock_guard<std::mutex> lk(S->mu);
    out->submitted = S->submitted;
    out->completed = S->completed;
    out->failed = S->failed;
    out->queued = S->queue.size();
    out->in_flight_requests = S->in_flight_requests;
    out->in_flight_bytes = S->in_flight_bytes;
    out->in_flight_bytes_high_water = S->in_flight_bytes_hwm;
    out->tickets_kept = S->tickets.size();
    return QM_OK;
}

}  /* extern "C" */
