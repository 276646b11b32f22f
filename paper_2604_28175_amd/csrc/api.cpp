// C ABI (strait.h): contexts, model instances, dual-priority submission, completion records.
//
// A submitted batch follows the paper's three steps (Section 3.2): input into the instance's
// pinned buffer and an asynchronous host-to-device copy on a copy stream; the kernel sequence
// on the compute stream that belongs to the batch's priority level (Section 3.1), made to wait
// for the copy through an event; the device-to-host copy of the result into pinned memory.
// Nothing synchronises with the host in between.  A small input whose compute stream has nothing
// else to do goes in on the compute stream itself: there is nothing to overlap with, and the
// hand-over between two streams takes about 20 us.  The copy kernels take the timestamps that
// Strait's predictor is fed (measured H2D time, measured kernel latency) and set the flags that say
// the result has arrived (elementwise.hip); the host polls those: the thread that waits for the
// batch, or the compute stream's completion thread when nobody waits yet.  Whoever sees the flags
// stamps the host completion time (Section 5.1: latency ends when the result is back in host
// memory) and hands the result over, a large one chunk by chunk while the rest is on the link.
#include <sched.h>
#include <time.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <functional>
#include <new>

#include "phases.hpp"
#include "runtime.hpp"

namespace strait {
const char* last_error();
}
using namespace strait;

#define HIP_TRY(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess) { set_error("%s: %s", #expr, hipGetErrorString(e_)); return STRAIT_E_HIP; } \
    } while (0)

struct strait_ctx : Context {};
struct strait_model : Model {};
struct strait_ticket_s : Ticket {};

static int64_t now_ns() {
    timespec ts;
    clock_gettime(CLOCK_MONOTONIC, &ts);
    return (int64_t)ts.tv_sec * 1000000000LL + ts.tv_nsec;
}

// Results of this size and more leave on a copy stream, beside the next batch's kernels (12.6 MB of a 64-sequence encoder batch:
// 0.24 ms of host link); below, the hand-over costs more than it hides.  The thread that completes the batch enqueues the copy when
// it sees the kernels done: a wait enqueued ahead would hold back whatever shares the copy stream's hardware queue (there are
// four of those, so two copy streams may be one queue), the next batches' inputs for instance.
static const size_t kOutOnCopyStream = 4u << 20;

// Whether a batch's result, on its way out, has another batch's kernels beside it: another compute stream's, or, on a copy stream, its own stream's next one's.
static bool others_run(Context* ctx, const Ticket* t) {
    for (size_t i = 0; i < ctx->workers.size(); ++i)
        if (ctx->workers[i]->outstanding.load(std::memory_order_acquire) > (i == t->worker && t->out_pending ? 1 : 0) && (i != t->worker || t->out_pending)) return true;
    return false;
}

// Enqueues the result's way out behind the kernel sequence on `s`.
static int enqueue_output(Model& m, Instance& in, Ticket* t, hipStream_t s) {
    const size_t bytes = m.out_bytes(t->batch);
    t->chunk_bytes = out_chunk_bytes(bytes);
    t->chunks = (unsigned)((bytes + t->chunk_bytes - 1) / t->chunk_bytes);
    t->out_pending = bytes >= kOutOnCopyStream;
    if (t->out_pending) return launch_stamp(in.ctl_dev, STAMP_K1, s, nullptr, nullptr, 0, t->seq);
    if (t->out_first < (int)m.ops.size()) return enqueue_classify_out(m, in, t->batch, t->out_first, s, t->hp, t->seq);
    return launch_copy_out(in.dev_out, in.pinned_out_dev, bytes, in.ctl_dev, in.counters + 1, t->seq, false, t->hp, others_run(m.ctx, t), s);
}

// A yielding low-priority batch (strait_ctx_set_lp_yield): its kernel sequence is enqueued by the stream's worker thread
// in segments of a few layers, at most two segments in flight, and before each further segment the thread waits while a
// high-priority batch is in flight on the GPU (at most kMaxYieldNs per segment, so that the wait always ends).  What
// the GPU runs beside a high-priority batch is then at most the rest of two short segments instead of a whole batch.
static const int64_t kMaxYieldNs = 5000000;
static int issue_in_segments(Context* ctx, StreamWorker* w, Ticket* t) {
    Model& m = *t->model;
    Instance& in = m.inst[t->instance];
    hipStream_t s = w->stream;
    const int n = t->out_first;
    int seg;
    { std::lock_guard<std::mutex> lk(ctx->mu); seg = ctx->lp_yield_layers > 0 ? ctx->lp_yield_layers : n; }
    if (hipStreamWaitEvent(s, in.ev_h2d, 0) != hipSuccess || launch_stamp(in.ctl_dev, STAMP_K0, s)) return STRAIT_E_HIP;
    int k = 0;
    for (int first = 0; first < n; first += seg, ++k) {
        if (k >= 1) {
            const int64_t t0 = now_ns();
            while (ctx->hp_in_flight.load(std::memory_order_acquire) > 0 && now_ns() - t0 < kMaxYieldNs) {
                timespec ts{0, 20000};
                nanosleep(&ts, nullptr);
            }
        }
        const int last = first + seg - 1 < n - 1 ? first + seg - 1 : n - 1;
        if (run_plan(m, in, t->batch, s, t->hp, last, false, first)) return STRAIT_E_HIP;
        if (hipEventRecord(in.ev_seg[k & 1], s) != hipSuccess) return STRAIT_E_HIP;
        if (k >= 1 && hipEventSynchronize(in.ev_seg[(k - 1) & 1]) != hipSuccess) return STRAIT_E_HIP;   // one segment of look-ahead
    }
    return enqueue_output(m, in, t, s);
}

// Polls until `there` is true, which something that is enqueued on `s` already makes it.  The wait ends: every few
// milliseconds the stream is asked whether it has failed, or has run dry without.  Not while a thread is submitting to it, that is holds
// its mutex: the stream may be recording a graph, which a query would spoil, and would itself be refused.
template <class There>
static int await(There there, hipStream_t s, std::mutex& submitting) {
    int64_t asked = 0;
    for (unsigned n = 1; !there(); ++n) {
        __builtin_ia32_pause();
        if (n & 255) continue;
        sched_yield();
        const int64_t now = now_ns();
        if (asked == 0) asked = now;
        if (now - asked < 5000000) continue;
        std::unique_lock<std::mutex> lk(submitting, std::try_to_lock);
        if (!lk.owns_lock()) continue;
        asked = now;
        const hipError_t e = hipStreamQuery(s);
        if (e == hipErrorNotReady) { (void)hipGetLastError(); continue; }
        if (e != hipSuccess || !there()) return STRAIT_E_HIP;
    }
    return 0;
}
// ... until the GPU has written `seq`.
static int await_flag(const uint32_t* flag, unsigned seq, hipStream_t s, std::mutex& submitting) {
    return await([=] { return __atomic_load_n(flag, __ATOMIC_ACQUIRE) == seq; }, s, submitting);
}

// Takes chunks of the result and copies each to the caller's buffer as it arrives, until none is left to take.  Two threads can be at it:
// one copies large results out of the pinned buffer at about 31 GB/s, the link brings 52.
static void copy_chunks(Ticket* t, Instance& in, hipStream_t s, std::mutex& submitting) {
    const size_t bytes = t->model->out_bytes(t->batch);
    const unsigned chunks = t->chunks;
    for (unsigned c; (c = t->chunk_next.fetch_add(1, std::memory_order_relaxed)) < chunks;) {
        const size_t at = (size_t)c * t->chunk_bytes;
        const int rc = await_flag(&in.ctl->flag[c], t->seq, s, submitting);
        if (c + 1 == chunks) t->t_last.store(now_ns(), std::memory_order_relaxed);
        if (rc) t->copy_status.store(rc, std::memory_order_relaxed);
        else memcpy((char*)t->host_out + at, (const char*)in.pinned_out + at, std::min<size_t>(t->chunk_bytes, bytes - at));
        t->chunk_done.fetch_add(1, std::memory_order_release);
    }
}

static hipStream_t output_stream(Context* ctx, const Ticket* t) { return t->out_pending ? ctx->copy[t->copy] : ctx->workers[t->worker]->stream; }
static std::mutex& output_mutex(Context* ctx, const Ticket* t) { return t->out_pending ? ctx->copy_mu[t->copy] : ctx->compute_mu[t->worker]; }

// Sees the result into the caller's buffer.  *done: host time at which its last part was seen in host memory.
static int await_result(Context* ctx, StreamWorker* w, Ticket* t, int64_t* done) {
    Instance& in = t->model->inst[t->instance];
    hipStream_t s = output_stream(ctx, t);
    if (t->out_pending) {
        if (await_flag(&in.ctl->k1_seq, t->seq, w->stream, ctx->compute_mu[t->worker])) return STRAIT_E_HIP;
        std::lock_guard<std::mutex> lk(ctx->copy_mu[t->copy]);
        ++ctx->copy_seq[t->copy];
        if (launch_copy_out(in.dev_out, in.pinned_out_dev, t->model->out_bytes(t->batch), in.ctl_dev, in.counters + 1, t->seq, true, t->hp, others_run(ctx, t), s)) return STRAIT_E_HIP;
    }
    if (t->chunks > 1) {
        std::lock_guard<std::mutex> lk(ctx->mu);
        t->chunks_coming.store(true, std::memory_order_release);
        ctx->cv_done.notify_all();
    }
    copy_chunks(t, in, s, output_mutex(ctx, t));
    while (t->chunk_done.load(std::memory_order_acquire) < t->chunks) __builtin_ia32_pause();   // the other thread's last memcpy
    *done = t->t_last.load(std::memory_order_relaxed);
    return t->copy_status.load(std::memory_order_relaxed);
}

// The time that the pieces of an input take on the link, `span` from `start` (host clock) to the end of the last, waits for the host's own
// copying between them left out: that of a first-in first-out link which is handed the pieces when this one was and ends when this one
// did, its rate found by bisection.  With `last`, the time of the last piece, its rate stands for all of them.
static float link_ms(const InputTiming& it, int64_t start, float span, float last) {
    double total = 0;
    for (int i = 0; i < it.pieces; ++i) total += (double)it.bytes[i];
    if (last > 0) return (float)(last * total / it.bytes[it.pieces - 1]);
    double lo = 0, hi = span;                          // time for all bytes
    for (int n = 0; it.pieces > 1 && n < 40; ++n) {
        const double mid = 0.5 * (lo + hi);
        double end = 0;
        for (int i = 0; i < it.pieces; ++i) end = std::max(end, (double)(it.handed[i] - start) * 1e-6) + mid * it.bytes[i] / total;
        if (end > span) hi = mid; else lo = mid;
    }
    return (float)hi;
}

// A batch's input does not count any longer on the copy streams that brought it.
static void leave_copy_streams(Context* ctx, const Ticket* t) {
    for (int i = 0; i < t->copies; ++i) ctx->copy_outstanding[(t->copy + i) % ctx->copy.size()].fetch_sub(1, std::memory_order_acq_rel);
    if (t->copies > 1 && t->prio == STRAIT_PRIO_LOW) ctx->low_in_parts.fetch_sub(1, std::memory_order_acq_rel);
}

// Sees a ticket that has left its stream's queue through to its end: result, record, completion.
static void complete_ticket(Context* ctx, StreamWorker* w, Ticket* t) {
    Instance& in = t->model->inst[t->instance];
    int status = 0;
    if (t->deferred) status = issue_in_segments(ctx, w, t);
    int64_t done = 0;
    if (!status) status = await_result(ctx, w, t, &done);
    if (!status && t->copies > 1) {                    // (see send_input)
        const size_t last = (t->copy + (t->input.pieces - 1) % 2) % ctx->copy.size();
        status = await([&] { return __atomic_load_n(&in.ctl->stamp[STAMP_PIECES + 1], __ATOMIC_ACQUIRE) != 0; }, ctx->copy[last], ctx->copy_mu[last]);
    }
    if (!done) done = now_ns();
    w->outstanding.fetch_sub(1, std::memory_order_acq_rel);
    leave_copy_streams(ctx, t);
    if (t->prio == STRAIT_PRIO_HIGH) ctx->hp_in_flight.fetch_sub(1, std::memory_order_acq_rel);
    if (!status) {
        const volatile uint64_t* st = in.ctl->stamp;
        auto ms = [&](uint64_t from, uint64_t to) { return (float)((double)(int64_t)(to - from) * ctx->ms_per_tick); };
        const volatile uint64_t* piece = st + STAMP_PIECES;
        const InputTiming& it = t->input;
        const uint64_t k0 = t->k0_stamped ? st[STAMP_K0] : piece[2 * it.pieces - 1];
        if (it.by_kernel) for (int i = 0; i < it.pieces; ++i) t->rec.h2d_ms += ms(piece[2 * i], piece[2 * i + 1]);
        else {
            // the transfer's start on the host's clock: from when a small result was seen, else when its first piece was handed over (earlier
            // than it started by the first launch's milliseconds, where it is the process's first)
            const int64_t start = t->chunks == 1 ? done - (int64_t)(1e6 * ms(piece[0], st[STAMP_DONE])) : it.handed[0];
            t->rec.h2d_ms = link_ms(it, start, ms(piece[0], piece[1]), it.last_timed ? ms(st[STAMP_LAST], piece[1]) : 0.f);
        }
        t->rec.kernel_ms = ms(k0, st[STAMP_K1]);
        t->rec.d2h_ms = ms(st[t->out_pending ? STAMP_D2H0 : STAMP_K1], st[STAMP_DONE]);
        t->rec.total_ms = ms(piece[0], st[STAMP_DONE]);
    }
    {
        std::lock_guard<std::mutex> lk(ctx->mu);
        t->rec.t_done_ns = done;
        t->status = status;
        t->done.store(true, std::memory_order_release);
        ctx->cv_done.notify_all();       // under the lock: the waiter may delete the ticket as soon as it sees it done
    }
}

static void worker_loop(Context* ctx, StreamWorker* w) {
    (void)hipSetDevice(ctx->device);
    for (;;) {
        Ticket* t = nullptr;
        {
            std::unique_lock<std::mutex> lk(ctx->mu);
            ctx->cv_work.wait(lk, [&] { return ctx->stop || !w->q.empty(); });
            if (w->q.empty()) return;           // stop requested and nothing left
            t = w->q.front();
            w->q.pop_front();
        }
        complete_ticket(ctx, w, t);
    }
}

extern "C" {

const char* strait_last_error(void) { return strait::last_error(); }
int32_t strait_version(void) { return 1; }

strait_status strait_ctx_create(const strait_ctx_desc* d, strait_ctx** out) {
    if (!d || !out) { set_error("ctx_create: null argument"); return STRAIT_E_INVALID; }
    if (d->n_hp < 1 || d->n_lp < 1 || d->n_copy < 1 || d->n_hp > STRAIT_MAX_STREAMS || d->n_lp > STRAIT_MAX_STREAMS ||
        d->n_copy > STRAIT_MAX_STREAMS) { set_error("ctx_create: stream counts must be in 1..%d", STRAIT_MAX_STREAMS); return STRAIT_E_INVALID; }
    int ndev = 0;
    HIP_TRY(hipGetDeviceCount(&ndev));
    if (d->device < 0 || d->device >= ndev) { set_error("ctx_create: device %d not present (%d devices)", d->device, ndev); return STRAIT_E_INVALID; }
    HIP_TRY(hipSetDevice(d->device));
    strait_ctx* c = new (std::nothrow) strait_ctx();
    if (!c) { set_error("out of host memory"); return STRAIT_E_NOMEM; }
    c->device = d->device;
    int khz = 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, d->device) != hipSuccess || khz <= 0) {
        delete c;
        set_error("ctx_create: the device's clock rate is not known");
        return STRAIT_E_HIP;
    }
    c->ms_per_tick = 1.0 / khz;
    for (int i = 0; i < d->n_hp; ++i) c->hp.push_back((hipStream_t)d->hp_streams[i]);
    for (int i = 0; i < d->n_lp; ++i) c->lp.push_back((hipStream_t)d->lp_streams[i]);
    for (int i = 0; i < d->n_copy; ++i) c->copy.push_back((hipStream_t)d->copy_streams[i]);
    for (size_t i = 0; i < c->hp.size() + c->lp.size(); ++i) {
        StreamWorker* w = new StreamWorker();
        w->stream = i < c->hp.size() ? c->hp[i] : c->lp[i - c->hp.size()];
        c->workers.push_back(w);
    }
    c->compute_mu.resize(c->workers.size());
    c->copy_mu.resize(c->copy.size());
    c->copy_seq.resize(c->copy.size(), 0);
    c->copy_outstanding.resize(c->copy.size());
    for (StreamWorker* w : c->workers) w->th = std::thread(worker_loop, (Context*)c, w);
    *out = c;
    return STRAIT_OK;
}

strait_status strait_ctx_destroy(strait_ctx* c) {
    if (!c) { set_error("ctx_destroy: null"); return STRAIT_E_INVALID; }
    {
        std::lock_guard<std::mutex> lk(c->mu);
        if (c->n_models > 0) { set_error("ctx_destroy: %d models still loaded", c->n_models); return STRAIT_E_BUSY; }
        c->stop = true;
    }
    c->cv_work.notify_all();
    for (StreamWorker* w : c->workers) { if (w->th.joinable()) w->th.join(); delete w; }
    delete c;
    return STRAIT_OK;
}

strait_status strait_ctx_set_wave_priority(strait_ctx* c, int32_t enabled) {
    if (!c) { set_error("ctx_set_wave_priority: null"); return STRAIT_E_INVALID; }
    std::lock_guard<std::mutex> lk(c->mu);
    c->wave_priority = enabled != 0;
    return STRAIT_OK;
}

strait_status strait_ctx_set_graphs(strait_ctx* c, int32_t enabled) {
    if (!c) { set_error("ctx_set_graphs: null"); return STRAIT_E_INVALID; }
    std::lock_guard<std::mutex> lk(c->mu);
    c->use_graphs = enabled != 0;
    return STRAIT_OK;
}

strait_status strait_ctx_set_h2d_kernel_limit(strait_ctx* c, int64_t max_bytes) {
    if (!c || max_bytes < 0) { set_error("ctx_set_h2d_kernel_limit: null context or negative size"); return STRAIT_E_INVALID; }
    std::lock_guard<std::mutex> lk(c->mu);
    c->h2d_kernel_limit = (size_t)max_bytes;
    return STRAIT_OK;
}

strait_status strait_ctx_set_pair_fusion(strait_ctx* c, int64_t min_pixels) {
    if (!c || min_pixels < 0) { set_error("ctx_set_pair_fusion: null context or negative size"); return STRAIT_E_INVALID; }
    std::lock_guard<std::mutex> lk(c->mu);
    c->pair_min_pixels = min_pixels;
    return STRAIT_OK;
}

strait_status strait_ctx_set_proj_fusion(strait_ctx* c, int64_t min_pixels) {
    if (!c || min_pixels < 0) { set_error("ctx_set_proj_fusion: null context or negative size"); return STRAIT_E_INVALID; }
    std::lock_guard<std::mutex> lk(c->mu);
    c->proj_min_pixels = min_pixels;
    return STRAIT_OK;
}

strait_status strait_ctx_set_lp_yield(strait_ctx* c, int32_t layers_per_segment) {
    if (!c || layers_per_segment < 0) { set_error("ctx_set_lp_yield: null context or negative segment length"); return STRAIT_E_INVALID; }
    std::lock_guard<std::mutex> lk(c->mu);
    c->lp_yield_layers = layers_per_segment;
    return STRAIT_OK;
}

strait_status strait_ctx_set_branch_streams(strait_ctx* c, int32_t enabled) {
    if (!c) { set_error("ctx_set_branch_streams: null"); return STRAIT_E_INVALID; }
    std::lock_guard<std::mutex> lk(c->mu);
    c->branch_streams = enabled != 0;
    return STRAIT_OK;
}

static int hp_flag(const Context* c, int prio) { return prio == STRAIT_PRIO_HIGH && c->wave_priority; }

// The kernel sequence of one batch on `s`: launched kernel by kernel, or, when the context asks for
// graphs, as one replay of the sequence captured for this (instance, batch, wave-priority) key.
// Only kernel launches are captured (no copies, events or memsets).  Only up to layer out_first, from
// which on the launch behind it computes them (enqueue_output).
// (With `lead`, layers 0..lead - 1 are enqueued already, part by part.)
static int run_batch(Model& m, Instance& in, int batch, hipStream_t s, int hp, int out_first, int lead) {
    if (out_first == 0) return 0;
    const bool cut = out_first < (int)m.ops.size();
    const int last = cut ? out_first - 1 : -1;
    if (lead > 0) return run_plan(m, in, batch, s, hp, last, false, lead, false, 0, batch);
    if (!m.ctx->use_graphs) return run_plan(m, in, batch, s, hp, last, false);
    const std::pair<int, int> key(batch, hp | (cut ? 2 : 0));
    auto it = in.graphs.find(key);
    if (it == in.graphs.end()) {
        if (in.warmed.insert(key).second) return run_plan(m, in, batch, s, hp, last, false);
        hipGraph_t g = nullptr;
        HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        const int rc = run_plan(m, in, batch, s, hp, last, false);
        const hipError_t e = hipStreamEndCapture(s, &g);
        if (rc || e != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            if (!rc) set_error("graph capture failed: %s", hipGetErrorString(e));
            return rc ? rc : STRAIT_E_HIP;
        }
        hipGraphExec_t ex = nullptr;
        const hipError_t ei = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (ei != hipSuccess) { set_error("graph instantiate failed: %s", hipGetErrorString(ei)); return STRAIT_E_HIP; }
        it = in.graphs.emplace(key, ex).first;
    }
    HIP_TRY(hipGraphLaunch(it->second, s));
    return 0;
}

static void free_instance(Instance& in) {
    if (in.pinned_in) (void)hipHostFree(in.pinned_in);
    if (in.pinned_out) (void)hipHostFree(in.pinned_out);
    if (in.dev_in) (void)hipFree(in.dev_in);
    if (in.dev_out) (void)hipFree(in.dev_out);
    if (in.dev_valid) (void)hipFree(in.dev_valid);
    if (in.splitk_ws) (void)hipFree(in.splitk_ws);
    for (float2* s : in.ln_stats) if (s) (void)hipFree(s);
    for (void* b : in.bufs) if (b) (void)hipFree(b);
    if (in.side) { (void)hipStreamSynchronize(in.side); (void)hipStreamDestroy(in.side); }
    if (in.ctl) (void)hipHostFree(in.ctl);
    if (in.counters) (void)hipFree(in.counters);
    hipEvent_t evs[5] = {in.ev_h2d, in.ev_fork, in.ev_join, in.ev_seg[0], in.ev_seg[1]};
    for (hipEvent_t e : evs) if (e) (void)hipEventDestroy(e);
    for (hipEvent_t e : in.layer_ev) if (e) (void)hipEventDestroy(e);
    for (auto& kv : in.graphs) (void)hipGraphExecDestroy(kv.second);
    in = Instance();
}

static void free_model(strait_model* m) {
    for (Instance& in : m->inst) free_instance(in);
    for (void* d : m->dev_allocs) (void)hipFree(d);
    if (m->fold_tmp) (void)hipFree(m->fold_tmp);
    delete m;
}

static const size_t COUNTER_BYTES = (2 + OUT_MAX_CHUNKS + 2) / 4 * 16;   // one for the input, one for the chunks, one per chunk; whole 16 bytes

static strait_status load_model(strait_ctx* c, const strait_model_desc* d, bool fold_layernorms, strait_model** out) {
    strait_model* m = new (std::nothrow) strait_model();
    if (!m) { set_error("out of host memory"); return STRAIT_E_NOMEM; }
    m->ctx = c;
    m->max_batch = d->max_batch;
    m->fold_layernorms = fold_layernorms;
    int rc = build_plan(*m, d->weights, d->weights_bytes);
    if (rc) { free_model(m); return rc; }
    m->inst.resize(d->n_instances);
    const size_t inb = (m->in_bytes(d->max_batch) + 255) / 256 * 256, outb = (m->out_bytes(d->max_batch) + 255) / 256 * 256;
    for (Instance& in : m->inst) {
        bool ok = hipHostMalloc(&in.pinned_in, inb + (size_t)d->max_batch * 4, hipHostMallocDefault) == hipSuccess &&
                  hipHostMalloc(&in.pinned_out, outb, hipHostMallocDefault) == hipSuccess &&
                  hipHostGetDevicePointer(&in.pinned_in_dev, in.pinned_in, 0) == hipSuccess &&
                  hipHostGetDevicePointer(&in.pinned_out_dev, in.pinned_out, 0) == hipSuccess &&
                  hipMalloc(&in.dev_in, inb) == hipSuccess && hipMalloc(&in.dev_out, outb) == hipSuccess &&
                  hipMalloc((void**)&in.dev_valid, (size_t)d->max_batch * 4 + 256) == hipSuccess &&
                  hipMalloc((void**)&in.splitk_ws, SPLITK_WS_BYTES) == hipSuccess;
        for (size_t i = 0; ok && i < 2 && m->ln_folds; ++i)
            ok = hipMalloc((void**)&in.ln_stats[i], (size_t)d->max_batch * m->seq * (m->hidden / 64) * sizeof(float2)) == hipSuccess;
        for (size_t i = 0; ok && i < m->buf_elems.size(); ++i) {
            void* b = nullptr;
            const size_t bytes = (m->buf_elems[i] * 2 * (size_t)d->max_batch + 255) / 256 * 256;
            ok = hipMalloc(&b, bytes) == hipSuccess;
            in.bufs.push_back(b);
        }
        ok = ok && hipHostMalloc((void**)&in.ctl, sizeof(HostControl), hipHostMallocDefault) == hipSuccess &&
             hipHostGetDevicePointer((void**)&in.ctl_dev, in.ctl, 0) == hipSuccess &&
             hipMalloc((void**)&in.counters, COUNTER_BYTES) == hipSuccess &&
             hipEventCreateWithFlags(&in.ev_h2d, hipEventDisableTiming) == hipSuccess &&
             hipEventCreateWithFlags(&in.ev_seg[0], hipEventDisableTiming) == hipSuccess &&
             hipEventCreateWithFlags(&in.ev_seg[1], hipEventDisableTiming) == hipSuccess &&
             hipStreamCreateWithFlags(&in.side, hipStreamNonBlocking) == hipSuccess &&      // default priority
             hipEventCreateWithFlags(&in.ev_fork, hipEventDisableTiming) == hipSuccess &&
             hipEventCreateWithFlags(&in.ev_join, hipEventDisableTiming) == hipSuccess;
        if (ok) {
            in.layer_ev.resize(m->ops.size() + 1, nullptr);
            for (hipEvent_t& e : in.layer_ev) ok = ok && hipEventCreate(&e) == hipSuccess;
        }
        if (!ok) {
            (void)hipGetLastError();
            set_error("model_load: allocating an instance (%zu B in, %zu B out, %zu activation buffers) failed", inb, outb, m->buf_elems.size());
            free_model(m);
            return STRAIT_E_NOMEM;
        }
        // The runtime sets a stream's hardware queue up at the first launch on it, which takes milliseconds:
        // do that here and not under the first batch that happens to use this instance's side stream.
        memset(in.ctl, 0, sizeof(HostControl));
        if (launch_fill_zero(in.counters, COUNTER_BYTES, in.side) != 0) { free_model(m); return STRAIT_E_HIP; }
        // valid lengths default to the full sequence
        if (m->arch == STRAIT_ARCH_ENCODER || m->arch == STRAIT_ARCH_VIT) {
            std::vector<int32_t> full(d->max_batch, m->seq);
            HIP_TRY(hipMemcpy(in.dev_valid, full.data(), full.size() * 4, hipMemcpyHostToDevice));
        }
    }
    if ((rc = finish_plan(*m))) { free_model(m); return rc; }
    HIP_TRY(hipDeviceSynchronize());
    {
        std::lock_guard<std::mutex> lk(c->mu);
        m->id = c->next_model_id++;
        c->n_models++;
    }
    *out = m;
    return STRAIT_OK;
}

strait_status strait_model_load(strait_ctx* c, const strait_model_desc* d, strait_model** out) {
    if (!c || !d || !out || !d->weights) { set_error("model_load: null argument"); return STRAIT_E_INVALID; }
    if (d->max_batch < 1 || d->max_batch > 4096 || d->n_instances < 1 || d->n_instances > 64) {
        set_error("model_load: max_batch must be in 1..4096 and n_instances in 1..64"); return STRAIT_E_INVALID;
    }
    HIP_TRY(hipSetDevice(c->device));
    // Folded LayerNorms need a second set of weights for the products behind them (half of a transformer's) and memory for statistics: a model that
    // fits without them only is loaded without them.
    strait_status rc = load_model(c, d, true, out);
    if (rc == STRAIT_E_NOMEM) {
        (void)hipGetLastError();
        rc = load_model(c, d, false, out);
    }
    if (rc) (void)hipGetLastError();      // reported here: the thread's next launch shall not find it
    return rc;
}

strait_status strait_model_free(strait_model* m) {
    if (!m) { set_error("model_free: null"); return STRAIT_E_INVALID; }
    {
        std::lock_guard<std::mutex> lk(m->mu);
        if (m->in_flight > 0) { set_error("model_free: %d batches in flight", m->in_flight); return STRAIT_E_BUSY; }
    }
    Context* c = m->ctx;
    (void)hipSetDevice(c->device);
    (void)hipDeviceSynchronize();
    free_model(m);
    std::lock_guard<std::mutex> lk(c->mu);
    c->n_models--;
    return STRAIT_OK;
}

strait_status strait_model_io(const strait_model* m, int32_t batch, size_t* in_bytes, size_t* out_bytes) {
    if (!m) { set_error("model_io: null"); return STRAIT_E_INVALID; }
    if (batch < 1 || batch > m->max_batch) { set_error("batch %d outside 1..%d", batch, m->max_batch); return STRAIT_E_BATCH; }
    if (in_bytes) *in_bytes = m->in_bytes(batch);
    if (out_bytes) *out_bytes = m->out_bytes(batch);
    return STRAIT_OK;
}

strait_status strait_model_info(const strait_model* m, int32_t* arch, int32_t* n_layers, int32_t* max_batch,
                                int32_t* n_instances, int32_t hyper[8]) {
    if (!m) { set_error("model_info: null"); return STRAIT_E_INVALID; }
    if (arch) *arch = m->arch;
    if (n_layers) *n_layers = (int32_t)m->ops.size();
    if (max_batch) *max_batch = m->max_batch;
    if (n_instances) *n_instances = (int32_t)m->inst.size();
    if (hyper) for (int i = 0; i < 8; ++i) hyper[i] = m->hyper[i];
    return STRAIT_OK;
}

strait_status strait_model_staging(const strait_model* m, int32_t instance, void** host_in, size_t* capacity) {
    if (!m || !host_in) { set_error("model_staging: null"); return STRAIT_E_INVALID; }
    if (instance < 0 || instance >= (int)m->inst.size()) { set_error("instance %d outside 0..%zu", instance, m->inst.size() - 1); return STRAIT_E_INVALID; }
    *host_in = m->inst[instance].pinned_in;
    if (capacity) *capacity = m->in_bytes(m->max_batch);
    return STRAIT_OK;
}

strait_status strait_model_layer(const strait_model* m, int32_t layer, strait_layer_info* out) {
    if (!m || !out) { set_error("model_layer: null"); return STRAIT_E_INVALID; }
    if (layer < 0 || layer >= (int)m->ops.size()) { set_error("layer %d outside 0..%zu", layer, m->ops.size() - 1); return STRAIT_E_INVALID; }
    *out = m->ops[layer].info;
    return STRAIT_OK;
}

static int check_call(strait_model* m, int instance, int prio, int batch) {
    if (!m) { set_error("null model"); return STRAIT_E_INVALID; }
    if (instance < 0 || instance >= (int)m->inst.size()) { set_error("instance %d outside 0..%zu", instance, m->inst.size() - 1); return STRAIT_E_INVALID; }
    if (prio != STRAIT_PRIO_HIGH && prio != STRAIT_PRIO_LOW) { set_error("priority must be STRAIT_PRIO_HIGH or STRAIT_PRIO_LOW"); return STRAIT_E_INVALID; }
    if (batch < 1 || batch > m->max_batch) { set_error("batch %d outside 1..%d", batch, m->max_batch); return STRAIT_E_BATCH; }
    return 0;
}

static hipStream_t compute_stream(Context* c, int prio, int instance) {
    return prio == STRAIT_PRIO_HIGH ? c->hp[instance % c->hp.size()] : c->lp[instance % c->lp.size()];
}

// Index of a compute stream in Context::workers / compute_mu (hp streams first, then lp).
static size_t compute_index(const Context* c, int prio, unsigned n) {
    return prio == STRAIT_PRIO_HIGH ? n % c->hp.size() : c->hp.size() + n % c->lp.size();
}

// Whether an input goes in by the copy kernel: inputs of serving-sized batches do (an asynchronous copy call of such a size now
// and then blocks its caller for milliseconds).
static bool input_by_kernel(const strait_model* m, int batch) {
    std::lock_guard<std::mutex> lk(m->ctx->mu);
    return m->in_bytes(batch) <= m->ctx->h2d_kernel_limit && (m->in_bytes(batch) & 3) == 0;
}
// The input (and the valid lengths) into the instance's pinned buffer and on to the device: through copy stream `ci`, or, with ci < 0, by
// kernel through `s`, whose mutex the caller holds.  An input that is not in the pinned buffer yet goes piece by piece, so that the
// host's copy of one piece and the link's of the one before go on together.  The link brings 52 GB/s, the host copies 75 from its caches
// and 31 from memory; each piece is half as large again as the one before it: few launches, and the first piece is soon on the way.  A batch of
// 1.5 MB: 374 us from submission to result in one piece, 355 in three.
// A piece by kernel takes its own stamps.  Between pieces that a copy engine brings, a stamp (or asking whether it has run dry) holds it
// up: 64 images of 224 x 224 at 2.05 ms, 40 us.  There the whole input is timed, and what the host's copying adds is known from when
// it handed the pieces over (link_ms).  That needs a stream with nothing else on it: an input that finds another batch's ahead goes in one
// piece, as the link has work meanwhile (`alone`), and once another's has come between, the rest goes as one with a start of its own.
// With `parts` (a staged input through copy engines), pieces of so many samples go through two copy streams in turn: what a record behind a piece holds its stream
// up by, 40 us, the other one's transfer fills.  Each is followed by in.ev_h2d and part_sent(its first sample, the sample behind its last); the valid lengths go ahead of them.
static int send_input(const strait_model* m, Instance& in, int batch, const void* host_in, const int32_t* valid_len, bool by_kernel, bool alone, int ci, hipStream_t s,
                      InputTiming* timing, const Parts& parts = Parts(), const std::function<int(int, int)>& part_sent = nullptr) {
    Context* c = m->ctx;
    const size_t inb = m->in_bytes(batch), off = (m->in_bytes(m->max_batch) + 255) / 256 * 256;
    const size_t lens = m->arch == STRAIT_ARCH_ENCODER ? (size_t)batch * 4 : 0;
    if (lens) {
        int32_t* pv = (int32_t*)((char*)in.pinned_in + off);
        for (int i = 0; i < batch; ++i) pv[i] = valid_len[i] < 0 ? 0 : (valid_len[i] > m->seq ? m->seq : valid_len[i]);
    }
    const void* lsrc = lens ? (const char*)in.pinned_in_dev + off : nullptr;
    void* ldst = lens ? in.dev_valid : nullptr;
    const bool staged = host_in == in.pinned_in;
    const bool part = parts.layers > 0;
    size_t piece = part ? m->in_bytes(parts.each) : staged ? inb : by_kernel ? 512u << 10 : alone ? 4u << 20 : inb;
    timing->by_kernel = by_kernel;
    timing->last_timed = false;
    unsigned seq[2] = {0, 0};                          // of this batch's previous piece on a stream
    const int first_ci = ci;
    int k = 0;
    for (size_t at = 0; at < inb; ++k) {
        size_t n = inb - at <= piece + piece / 2 || k == MAX_PIECES - 1 ? inb - at : piece;
        const int turn = part ? k & 1 : 0;
        if (part) {
            if (k == 0) n = m->in_bytes(parts.first);
            ci = (first_ci + turn) % (int)c->copy.size();
            s = c->copy[ci];
        }
        if (!staged) memcpy((char*)in.pinned_in + at, (const char*)host_in + at, n);
        std::unique_lock<std::mutex> lk;
        if (ci >= 0) lk = std::unique_lock<std::mutex>(c->copy_mu[ci]);
        if (!by_kernel && k > turn && c->copy_seq[ci] != seq[turn]) {
            timing->last_timed = true;
            if (at + n < inb) {
                lk.unlock();
                if (!staged) memcpy((char*)in.pinned_in + at + n, (const char*)host_in + at + n, inb - at - n);
                n = inb - at;
                lk.lock();
            }
        }
        const bool last = at + n == inb;
        timing->pieces = k + 1;
        timing->handed[k] = now_ns();
        timing->bytes[k] = n;
        if (ci >= 0) seq[turn] = ++c->copy_seq[ci];
        if (by_kernel) {
            if (launch_copy_in((const char*)in.pinned_in_dev + at, (char*)in.dev_in + at, n, lsrc, ldst, last ? lens : 0, in.ctl_dev, in.counters, k, s))
                return STRAIT_E_HIP;
        } else {
            if (k == 0 && launch_stamp(in.ctl_dev, STAMP_PIECES, s, lsrc, ldst, part ? lens : 0)) return STRAIT_E_HIP;
            if (timing->last_timed && launch_stamp(in.ctl_dev, STAMP_LAST, s)) return STRAIT_E_HIP;
            HIP_TRY(hipMemcpyAsync((char*)in.dev_in + at, (const char*)in.pinned_in + at, n, hipMemcpyHostToDevice, s));
            if (part) HIP_TRY(hipEventRecord(in.ev_h2d, s));
            // Of parts, nothing on the compute stream waits for this stamp (a launch between a transfer and the event behind it is 20 us of ViT's 3640, 64 images): who completes
            // the batch does, before the record is read and the instance given to another batch.
            if (part && last) __atomic_store_n(&in.ctl->stamp[STAMP_PIECES + 1], 0, __ATOMIC_RELAXED);
            if (last && launch_stamp(in.ctl_dev, STAMP_PIECES + 1, s, lsrc, ldst, part ? 0 : lens)) return STRAIT_E_HIP;
        }
        if (part) {
            lk.unlock();
            const int rc = part_sent((int)(at / m->in_bytes(1)), (int)((at + n) / m->in_bytes(1)));
            if (rc) return rc;
        } else piece += piece / 2 & ~(size_t)15;
        at += n;
    }
    return 0;
}

strait_status strait_submit(strait_model* m, strait_priority prio, int32_t batch, const void* host_in,
                            const int32_t* valid_len, void* host_out, strait_ticket* ticket) {
    const int64_t t_enq = now_ns();
    int rc = check_call(m, 0, prio, batch);
    if (rc) return rc;
    if (!host_in || !host_out || !ticket) { set_error("submit: null argument"); return STRAIT_E_INVALID; }
    if (m->arch == STRAIT_ARCH_ENCODER && !valid_len) { set_error("submit: the encoder needs valid_len"); return STRAIT_E_INVALID; }
    Context* c = m->ctx;
    int idx = -1;
    {
        std::lock_guard<std::mutex> lk(m->mu);
        int staged = -1;                              // input already in an instance's pinned buffer?
        for (size_t i = 0; i < m->inst.size(); ++i)
            if (host_in == m->inst[i].pinned_in) staged = (int)i;
        if (staged >= 0) {
            if (m->inst[staged].busy) { set_error("submit: instance %d, whose staging buffer was given, is busy", staged); return STRAIT_E_BUSY; }
            idx = staged;
        } else {
            for (size_t i = 0; i < m->inst.size(); ++i)
                if (!m->inst[i].busy) { idx = (int)i; break; }
        }
        if (idx < 0) { set_error("submit: all %zu instances busy", m->inst.size()); return STRAIT_E_BUSY; }
        m->inst[idx].busy = true;
        m->in_flight++;
    }
    auto release = [&]() { std::lock_guard<std::mutex> lk(m->mu); m->inst[idx].busy = false; m->in_flight--; };
    strait_ticket_s* t = new (std::nothrow) strait_ticket_s();
    if (!t) { release(); set_error("out of host memory"); return STRAIT_E_NOMEM; }
    Instance& in = m->inst[idx];
    unsigned si, ci;
    {
        std::lock_guard<std::mutex> lk(c->mu);
        si = prio == STRAIT_PRIO_HIGH ? c->n_hp_sub++ : c->n_lp_sub++;
        ci = c->n_copy_sub++;
    }
    const size_t widx = compute_index(c, prio, si);
    const size_t cidx = ci % c->copy.size();
    StreamWorker* w = c->workers[widx];
    hipStream_t s = w->stream;
    hipStream_t cs = c->copy[cidx];
    rc = hipSetDevice(c->device) == hipSuccess ? 0 : STRAIT_E_HIP;
    const bool by_kernel = input_by_kernel(m, batch);
    t->model = m; t->instance = idx; t->prio = prio; t->batch = batch; t->host_out = host_out; t->worker = widx;
    t->copy = cidx;
    if (++in.seq == 0) ++in.seq;         // 0: no number
    t->seq = in.seq;
    t->rec.model_id = m->id; t->rec.priority = prio; t->rec.batch = batch; t->rec.instance = idx;
    t->rec.t_enqueue_ns = t_enq;
    bool yielding;
    { std::lock_guard<std::mutex> lk(c->mu); yielding = prio == STRAIT_PRIO_LOW && c->lp_yield_layers > 0; }
    t->hp = hp_flag(c, prio);
    t->out_first = classify_out_first(*m, batch);
    if (prio == STRAIT_PRIO_HIGH) c->hp_in_flight.fetch_add(1, std::memory_order_acq_rel);
    int lead = 0;                        // layers that are computed part by part, as the input comes in
    std::unique_lock<std::mutex> slk(c->compute_mu[widx], std::defer_lock);
    auto h2d_on_copy_stream = [&]() {
        const bool alone = c->copy_outstanding[cidx].fetch_add(1, std::memory_order_acq_rel) == 0;
        t->copies = 1;
        // A large input that is staged and that nothing else is on its way beside: the first layers of each part run while the next part is on the link, where 64 images of
        // 224 x 224 are 365 us.  In one piece (replayed from a graph) and in parts: MobileNetV2 64 images 940 -> 873 us, 128 images 1625 -> 1463, 31 images 601 -> 588; ViT 64 images 3700 ->
        // 3608, 45 images 2834 -> 2786; VGG-19 64 images 3161 -> 3099; encoder 64 sequences 2848 -> 2799, 100 sequences 4084 -> 3939.
        // An input that is not staged waits for the host's copying, which these launches would hold up; a captured kernel sequence is one piece.
        Parts parts;
        if (host_in == in.pinned_in && !yielding && !by_kernel && !c->use_graphs && !InputFirst::wanted() && c->copy.size() > 1 && w->outstanding.load(std::memory_order_acquire) == 0)
            parts = plan_parts(*m, batch, t->out_first);
        if (parts.layers) {
            std::atomic<int>& second = c->copy_outstanding[(cidx + 1) % c->copy.size()];
            second.fetch_add(1, std::memory_order_acq_rel);     // (before looking: of two batches that come at the same time at most one goes in parts)
            int others = -2;
            for (const auto& n : c->copy_outstanding) others += n.load(std::memory_order_acquire);
            if (others == 0) {
                lead = parts.layers;
                t->copies = 2;
                if (prio == STRAIT_PRIO_LOW) c->low_in_parts.fetch_add(1, std::memory_order_acq_rel);
                return send_input(m, in, batch, host_in, valid_len, false, true, (int)cidx, cs, &t->input, parts, [&](int first, int end) {
                    if (!slk.owns_lock()) slk.lock();
                    if (hipStreamWaitEvent(s, in.ev_h2d, 0) != hipSuccess) return (int)STRAIT_E_HIP;
                    if (first == 0 && launch_stamp(in.ctl_dev, STAMP_K0, s)) return (int)STRAIT_E_HIP;
                    const int r = run_plan(*m, in, end - first, s, t->hp, lead - 1, false, 0, false, first, batch);
                    if (end < batch) slk.unlock();
                    return r;
                });
            }
            second.fetch_sub(1, std::memory_order_acq_rel);
        }
        int r = send_input(m, in, batch, host_in, valid_len, by_kernel, alone, (int)cidx, cs, &t->input);
        std::lock_guard<std::mutex> lk(c->copy_mu[cidx]);
        if (!r) r = hipEventRecord(in.ev_h2d, cs) == hipSuccess ? 0 : STRAIT_E_HIP;
        return r;
    };
    if (yielding) {
        // the stream's worker thread enqueues the kernels, segment by segment (issue_in_segments)
        t->deferred = true;
        t->k0_stamped = true;
        if (!rc) rc = h2d_on_copy_stream();
        if (!rc) {
            t->rec.t_issued_ns = now_ns();
            std::lock_guard<std::mutex> lk(c->mu);
            w->outstanding.fetch_add(1, std::memory_order_acq_rel);
            w->q.push_back(t);
        }
    } else {
        // A small input goes in on an idle compute stream itself; otherwise it travels beside the batches ahead of it (enqueued
        // before this stream's mutex is taken, so that a batch that is being issued does not hold its transfer up).  With one copy
        // stream every input goes through it, so that transfers stay first-in first-out.  Where a low-priority batch's parts, all of which are
        // enqueued at once, lie on two copy streams, a high-priority input goes in behind its own level's batches and not behind those parts: eight images of ResNet-50
        // beside 128 of MobileNetV2 at low priority, submitted while eight images before them are computed, 1009 -> 847 us (788 and 793 once the parts are through).
        bool in_line = false;
        const bool past_parts = prio == STRAIT_PRIO_HIGH && c->low_in_parts.load(std::memory_order_acquire) > 0;
        if (by_kernel && c->copy.size() > 1 && (past_parts || w->outstanding.load(std::memory_order_acquire) == 0)) {
            slk.lock();
            in_line = past_parts || w->outstanding.load(std::memory_order_acquire) == 0;
        }
        if (in_line) {
            if (!rc) rc = send_input(m, in, batch, host_in, valid_len, true, true, -1, s, &t->input);
        } else {
            if (!rc) rc = h2d_on_copy_stream();
            if (!slk.owns_lock()) slk.lock();
            if (!rc && !lead) rc = hipStreamWaitEvent(s, in.ev_h2d, 0) == hipSuccess ? 0 : STRAIT_E_HIP;
            if (!rc && !lead) rc = launch_stamp(in.ctl_dev, STAMP_K0, s) ? STRAIT_E_HIP : 0;
            t->k0_stamped = true;
        }
        if (!rc) rc = run_batch(*m, in, batch, s, t->hp, t->out_first, lead);
        if (!rc) rc = enqueue_output(*m, in, t, s);
        if (!rc) {
            t->rec.t_issued_ns = now_ns();
            std::lock_guard<std::mutex> lk(c->mu);          // tickets join the worker's queue in stream order
            w->outstanding.fetch_add(1, std::memory_order_acq_rel);
            w->q.push_back(t);
        }
    }
    if (slk.owns_lock()) slk.unlock();
    if (rc) {
        if (prio == STRAIT_PRIO_HIGH) c->hp_in_flight.fetch_sub(1, std::memory_order_acq_rel);
        leave_copy_streams(c, t);
        if (rc == STRAIT_E_HIP && !strait::last_error()[0]) set_error("submit: a HIP call failed");
        (void)hipStreamSynchronize(s);
        for (hipStream_t copy : c->copy) (void)hipStreamSynchronize(copy);
        release();
        delete t;
        return rc;
    }
    c->cv_work.notify_all();
    *ticket = t;
    return STRAIT_OK;
}

strait_status strait_poll(strait_ticket t, int32_t* done) {
    if (!t || !done) { set_error("poll: null argument"); return STRAIT_E_INVALID; }
    *done = t->done.load(std::memory_order_acquire) ? 1 : 0;
    return STRAIT_OK;
}

strait_status strait_wait(strait_ticket t, strait_record* rec) {
    if (!t) { set_error("wait: null ticket"); return STRAIT_E_INVALID; }
    Model* m = t->model;
    Context* c = m->ctx;
    StreamWorker* w = c->workers[t->worker];
    // The next result of its stream is fetched by the thread that waits for it (no hand-over between threads); while another
    // thread is at it, look on for a while before going to sleep (a wake-up takes as long as some batches).
    bool mine = false;
    {
        std::lock_guard<std::mutex> lk(c->mu);
        if (!w->q.empty() && w->q.front() == t && !t->deferred) { w->q.pop_front(); mine = true; }
    }
    if (mine) {
        (void)hipSetDevice(c->device);
        complete_ticket(c, w, t);
    } else {
        auto can_help = [&] { return t->chunks_coming.load(std::memory_order_acquire) && t->chunk_next.load(std::memory_order_relaxed) < t->chunks; };
        bool done = false;
        while (!done) {
            const int64_t t0 = now_ns();
            while (!t->done.load(std::memory_order_acquire) && !can_help() && now_ns() - t0 < 500000)
                for (int i = 0; i < 32; ++i) __builtin_ia32_pause();
            {
                std::unique_lock<std::mutex> lk(c->mu);
                c->cv_done.wait(lk, [&] { return t->done.load(std::memory_order_acquire) || can_help(); });
                done = t->done.load(std::memory_order_acquire);
            }
            if (!done) copy_chunks(t, m->inst[t->instance], output_stream(c, t), output_mutex(c, t));
        }
    }
    if (rec) *rec = t->rec;
    const int status = t->status;
    {
        std::lock_guard<std::mutex> lk(m->mu);
        m->inst[t->instance].busy = false;
        m->in_flight--;
    }
    delete t;
    if (status) { set_error("wait: the batch failed on the device"); return status; }
    return STRAIT_OK;
}

strait_status strait_copy_in(strait_model* m, int32_t instance, strait_priority prio, int32_t batch,
                             const void* host_in, const int32_t* valid_len) {
    int rc = check_call(m, instance, prio, batch);
    if (rc) return rc;
    if (!host_in) { set_error("copy_in: null input"); return STRAIT_E_INVALID; }
    if (m->arch == STRAIT_ARCH_ENCODER && !valid_len) { set_error("copy_in: the encoder needs valid_len"); return STRAIT_E_INVALID; }
    Context* c = m->ctx;
    HIP_TRY(hipSetDevice(c->device));
    Instance& in = m->inst[instance];
    const size_t ci = (size_t)instance % c->copy.size();
    InputTiming timing;
    if ((rc = send_input(m, in, batch, host_in, valid_len, input_by_kernel(m, batch), true, (int)ci, c->copy[ci], &timing))) return rc;
    {
        std::lock_guard<std::mutex> lk(c->copy_mu[ci]);
        HIP_TRY(hipEventRecord(in.ev_h2d, c->copy[ci]));
    }
    std::lock_guard<std::mutex> slk(c->compute_mu[compute_index(c, prio, (unsigned)instance)]);
    HIP_TRY(hipStreamWaitEvent(compute_stream(c, prio, instance), in.ev_h2d, 0));
    return STRAIT_OK;
}

strait_status strait_run(strait_model* m, int32_t instance, strait_priority prio, int32_t batch) {
    int rc = check_call(m, instance, prio, batch);
    if (rc) return rc;
    HIP_TRY(hipSetDevice(m->ctx->device));
    std::lock_guard<std::mutex> slk(m->ctx->compute_mu[compute_index(m->ctx, prio, (unsigned)instance)]);
    return run_batch(*m, m->inst[instance], batch, compute_stream(m->ctx, prio, instance), hp_flag(m->ctx, prio), (int)m->ops.size(), 0);
}

strait_status strait_copy_out(strait_model* m, int32_t instance, strait_priority prio, int32_t batch, void* host_out) {
    int rc = check_call(m, instance, prio, batch);
    if (rc) return rc;
    if (!host_out) { set_error("copy_out: null output"); return STRAIT_E_INVALID; }
    Instance& in = m->inst[instance];
    hipStream_t s = compute_stream(m->ctx, prio, instance);
    HIP_TRY(hipSetDevice(m->ctx->device));
    HIP_TRY(hipMemcpyAsync(in.pinned_out, in.dev_out, m->out_bytes(batch), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    memcpy(host_out, in.pinned_out, m->out_bytes(batch));
    return STRAIT_OK;
}

strait_status strait_sync(strait_model* m, int32_t instance, strait_priority prio) {
    int rc = check_call(m, instance, prio, 1);
    if (rc) return rc;
    HIP_TRY(hipSetDevice(m->ctx->device));
    HIP_TRY(hipStreamSynchronize(compute_stream(m->ctx, prio, instance)));
    return STRAIT_OK;
}

strait_status strait_run_timed(strait_model* m, int32_t instance, strait_priority prio, int32_t batch, float* layer_ms) {
    int rc = check_call(m, instance, prio, batch);
    if (rc) return rc;
    if (!layer_ms) { set_error("run_timed: null output"); return STRAIT_E_INVALID; }
    Instance& in = m->inst[instance];
    hipStream_t s = compute_stream(m->ctx, prio, instance);
    HIP_TRY(hipSetDevice(m->ctx->device));
    rc = run_plan(*m, in, batch, s, hp_flag(m->ctx, prio), -1, true);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(s));
    for (size_t i = 0; i < m->ops.size(); ++i) {
        HIP_TRY(hipEventElapsedTime(&layer_ms[i], in.layer_ev[i], in.layer_ev[i + 1]));
        if (in.layer_skipped[i]) layer_ms[i] = 0.f;    // its time is in the launch that computed it (between its events: nothing)
    }
    return STRAIT_OK;
}

strait_status strait_read_activation(strait_model* m, int32_t instance, int32_t layer, int32_t batch, void* host_out,
                                     size_t bytes, size_t* needed) {
    int rc = check_call(m, instance, STRAIT_PRIO_LOW, batch);
    if (rc) return rc;
    if (layer < 0 || layer >= (int)m->ops.size()) { set_error("layer %d outside 0..%zu", layer, m->ops.size() - 1); return STRAIT_E_INVALID; }
    const Op& op = m->ops[layer];
    if (op.out < 0) { set_error("layer %d ('%s') writes to the output buffer; use copy_out", layer, op.name.c_str()); return STRAIT_E_INVALID; }
    const size_t need = (size_t)batch * op.P * op.Q * op.K * 2;
    if (needed) *needed = need;
    if (!host_out) return STRAIT_OK;
    if (bytes != need) { set_error("read_activation: layer '%s' holds %zu bytes for batch %d, caller gave %zu", op.name.c_str(), need, batch, bytes); return STRAIT_E_INVALID; }
    Instance& in = m->inst[instance];
    hipStream_t s = compute_stream(m->ctx, STRAIT_PRIO_LOW, instance);
    HIP_TRY(hipSetDevice(m->ctx->device));
    rc = run_plan(*m, in, batch, s, 0, layer, false, 0, true);     // re-run the prefix: later layers reuse buffers
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(s));
    HIP_TRY(hipMemcpy(host_out, in.bufs[op.out], need, hipMemcpyDeviceToHost));
    return STRAIT_OK;
}

// ---- kernel-level entry points -----------------------------------------------------------------

// Not while the stream records a graph: the launch is then one that needs no workspace.
static bool may_allocate(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st == hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

static int conv2d_params(ConvParams& p, int32_t N, int32_t H, int32_t W, int32_t C, int32_t K, int32_t R, int32_t S, int32_t stride, int32_t pad,
                         int32_t act, int32_t out_f32) {
    if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || K <= 0 || R <= 0 || S <= 0 || stride <= 0 || pad < 0 ||
        H + 2 * pad < R || W + 2 * pad < S) { set_error("conv2d: invalid shape"); return STRAIT_E_SHAPE; }
    const int P = (H + 2 * pad - R) / stride + 1, Q = (W + 2 * pad - S) / stride + 1;
    if ((long long)N * P * Q > 0x7fffffffLL || (long long)R * S * C > 0x7fffffffLL) { set_error("conv2d: too large"); return STRAIT_E_SHAPE; }
    p.M = N * P * Q; p.PQ = P * Q; p.Q = Q; p.H = H; p.W = W; p.C = C; p.R = R; p.S = S;
    p.stride_h = p.stride_w = stride; p.pad_h = p.pad_w = pad;
    p.sN = (long long)H * W * C; p.sH = W * C; p.sW = C;
    p.Kg = R * S * C; p.ldw = (p.Kg + 7) / 8 * 8; p.Cout = K; p.ldy = K; p.act = act; p.out_f32 = out_f32;
    return 0;
}

const char* strait_k_conv2d_kernel(int32_t N, int32_t H, int32_t W, int32_t C, int32_t K, int32_t R, int32_t S, int32_t stride, int32_t pad,
                                   int32_t act, int32_t res, int32_t out_f32) {
    ConvParams p{};
    if (conv2d_params(p, N, H, W, C, K, R, S, stride, pad, act, out_f32)) return nullptr;
    half_t* const some = reinterpret_cast<half_t*>(256);        // any aligned address: nothing is launched
    p.x = p.w = some; p.y = some; p.res = res ? some : nullptr; p.ws = (float*)some; p.ws_bytes = SPLITK_WS_BYTES;
    return conv_kernel_name(p);
}

strait_status strait_k_conv2d(void* stream, const void* x, int32_t N, int32_t H, int32_t W, int32_t C,
                              const void* w_krsc, const float* bias, int32_t K, int32_t R, int32_t S, int32_t stride,
                              int32_t pad, int32_t act, const void* res, void* y, int32_t out_f32, int32_t hp) {
    ConvParams p{};
    const int bad = conv2d_params(p, N, H, W, C, K, R, S, stride, pad, act, out_f32);
    if (bad) return bad;
    p.x = (const half_t*)x; p.bias = bias; p.res = (const half_t*)res; p.y = y; p.hp = hp;
    void* tmp = nullptr;
    if (p.Kg % 8 == 0) p.w = (const half_t*)w_krsc;
    else {
        // rows padded with zeros to a multiple of 8 elements, as the kernel's 16-byte weight loads need
        HIP_TRY(hipMalloc(&tmp, (size_t)K * p.ldw * 2));
        hipError_t e = hipMemsetAsync(tmp, 0, (size_t)K * p.ldw * 2, (hipStream_t)stream);
        if (e == hipSuccess) e = hipMemcpy2DAsync(tmp, (size_t)p.ldw * 2, w_krsc, (size_t)p.Kg * 2, (size_t)p.Kg * 2, K, hipMemcpyDeviceToDevice, (hipStream_t)stream);
        if (e != hipSuccess) { (void)hipFree(tmp); set_error("conv2d: padding the weights failed: %s", hipGetErrorString(e)); return STRAIT_E_HIP; }
        p.w = (const half_t*)tmp;
    }
    // a long reduction for few outputs may be split into slabs, which needs an fp32 workspace
    void* ws = nullptr;
    if (may_allocate((hipStream_t)stream) && conv_workspace_bytes(p, SPLITK_WS_BYTES)) {
        if (hipMalloc(&ws, SPLITK_WS_BYTES) != hipSuccess) { (void)hipGetLastError(); ws = nullptr; }
        p.ws = (float*)ws; p.ws_bytes = ws ? SPLITK_WS_BYTES : 0;
    }
    int rc = launch_conv(p, (hipStream_t)stream);
    if (tmp || ws) { (void)hipStreamSynchronize((hipStream_t)stream); if (tmp) (void)hipFree(tmp); if (ws) (void)hipFree(ws); }
    return rc;
}

strait_status strait_k_conv1x1_proj(void* stream, const void* x, int32_t N, int32_t P, int32_t Q, int32_t C, const void* x2,
                                    int32_t H2, int32_t W2, int32_t K2, int32_t stride2, const void* w, const float* bias,
                                    int32_t Cout, int32_t act, void* y, int32_t hp) {
    if (N <= 0 || P <= 0 || Q <= 0 || C <= 0 || K2 <= 0 || Cout <= 0 || stride2 <= 0 || H2 <= 0 || W2 <= 0 ||
        (long long)(P - 1) * stride2 >= H2 || (long long)(Q - 1) * stride2 >= W2 || (long long)N * P * Q > 0x7fffffffLL) {
        set_error("conv1x1_proj: invalid shape (every output pixel needs its pixel of the second tensor)"); return STRAIT_E_SHAPE;
    }
    if (!x2) { set_error("conv1x1_proj: x2 is required"); return STRAIT_E_INVALID; }
    ConvParams p{};
    p.x = (const half_t*)x; p.w = (const half_t*)w; p.bias = bias; p.y = y;
    p.M = N * P * Q; p.PQ = P * Q; p.Q = Q; p.H = P; p.W = Q; p.C = C; p.R = 1; p.S = 1;
    p.stride_h = p.stride_w = 1; p.pad_h = p.pad_w = 0;
    p.sN = (long long)P * Q * C; p.sH = Q * C; p.sW = C;
    p.x2 = (const half_t*)x2; p.K2 = K2; p.stride2 = stride2; p.sN2 = (long long)H2 * W2 * K2; p.sH2 = W2 * K2; p.sW2 = K2;
    p.Kg = C + K2; p.ldw = C + K2; p.Cout = Cout; p.ldy = Cout; p.act = act; p.hp = hp;
    return launch_conv(p, (hipStream_t)stream);
}

strait_status strait_k_gemm(void* stream, const void* x, const void* w, const float* bias, int32_t M, int32_t N,
                            int32_t K, int32_t act, const void* res, void* y, int32_t out_f32, int32_t hp) {
    if (M <= 0 || N <= 0 || K <= 0 || K % 8 != 0) { set_error("gemm: needs positive sizes and K %% 8 == 0"); return STRAIT_E_SHAPE; }
    ConvParams p{};
    p.x = (const half_t*)x; p.w = (const half_t*)w; p.bias = bias; p.res = (const half_t*)res; p.y = y;
    p.M = M; p.PQ = 1; p.Q = 1; p.H = 1; p.W = 1; p.C = K; p.R = 1; p.S = 1;
    p.stride_h = p.stride_w = 1; p.pad_h = p.pad_w = 0;
    p.sN = K; p.sH = K; p.sW = K; p.Kg = K; p.ldw = K; p.Cout = N; p.ldy = N; p.act = act; p.out_f32 = out_f32; p.hp = hp;
    void* ws = nullptr;
    if (may_allocate((hipStream_t)stream) && conv_workspace_bytes(p, SPLITK_WS_BYTES)) {
        if (hipMalloc(&ws, SPLITK_WS_BYTES) != hipSuccess) { (void)hipGetLastError(); ws = nullptr; }
        p.ws = (float*)ws; p.ws_bytes = ws ? SPLITK_WS_BYTES : 0;
    }
    int rc = launch_conv(p, (hipStream_t)stream);
    if (ws) { (void)hipStreamSynchronize((hipStream_t)stream); (void)hipFree(ws); }
    return rc;
}

strait_status strait_k_gemm_ln(void* stream, const void* x, const void* w, const float* bias, const void* res, int32_t M, int32_t N, int32_t K,
                               int32_t act, const float* ln_stats, const float* ln_csum, const float* ln_g, const float* ln_b, float ln_eps, void* y,
                               float* stats_out, int32_t hp) {
    if (M <= 0 || N <= 0 || K <= 0) { set_error("gemm_ln: needs positive sizes"); return STRAIT_E_SHAPE; }
    ConvParams p{};
    p.x = (const half_t*)x; p.w = (const half_t*)w; p.bias = bias; p.res = (const half_t*)res; p.y = y;
    p.M = M; p.PQ = 1; p.Q = 1; p.H = 1; p.W = 1; p.C = K; p.R = 1; p.S = 1;
    p.stride_h = p.stride_w = 1;
    p.sN = K; p.sH = K; p.sW = K; p.Kg = K; p.ldw = K; p.Cout = N; p.ldy = N; p.act = act; p.hp = hp;
    p.ln_stats = (const float2*)ln_stats; p.ln_csum = ln_csum; p.ln_g = ln_g; p.ln_b = ln_b; p.ln_eps = ln_eps; p.stats_out = (float2*)stats_out;
    return launch_gemm_ln(p, (hipStream_t)stream);
}

strait_status strait_k_fold_layernorm(void* stream, const void* w, const float* b, const float* gamma, const float* beta, int32_t N, int32_t K,
                                      void* w_out, float* csum, float* b_out) {
    return launch_fold_layernorm((const half_t*)w, b, gamma, beta, N, K, (half_t*)w_out, csum, b_out, nullptr, (hipStream_t)stream);
}

strait_status strait_k_pointwise_pair(void* stream, const void* x, const void* w3, const float* b3, const void* res, void* y,
                                      const void* w1, const float* b1, void* z, int32_t M, int32_t K1, int32_t N1, int32_t N2,
                                      int32_t act1, int32_t act2, int32_t hp) {
    PairParams p{};
    p.x = (const half_t*)x; p.w3 = (const half_t*)w3; p.b3 = b3; p.res = (const half_t*)res; p.y = (half_t*)y;
    p.w1 = (const half_t*)w1; p.b1 = b1; p.z = (half_t*)z;
    p.M = M; p.K1 = K1; p.N1 = N1; p.N2 = N2; p.act1 = act1; p.act2 = act2; p.hp = hp;
    return launch_pointwise_pair(p, (hipStream_t)stream);
}

strait_status strait_k_pointwise_pair_proj(void* stream, const void* x, const void* x2, const void* w3, const float* b3, void* y,
                                           const void* w1, const float* b1, void* z, int32_t M, int32_t K1, int32_t K2, int32_t N1,
                                           int32_t N2, int32_t act1, int32_t act2, int32_t hp) {
    if (!x2) { set_error("pointwise pair with projection: x2 is required"); return STRAIT_E_INVALID; }
    PairParams p{};
    p.x = (const half_t*)x; p.x2 = (const half_t*)x2; p.w3 = (const half_t*)w3; p.b3 = b3; p.y = (half_t*)y;
    p.w1 = (const half_t*)w1; p.b1 = b1; p.z = (half_t*)z;
    p.M = M; p.K1 = K1; p.K2 = K2; p.N1 = N1; p.N2 = N2; p.act1 = act1; p.act2 = act2; p.hp = hp;
    return launch_pointwise_pair(p, (hipStream_t)stream);
}

strait_status strait_k_dwconv3x3(void* stream, const void* x, int32_t N, int32_t H, int32_t W, int32_t C,
                                 const void* w_rsc, const float* bias, int32_t stride, int32_t act, void* y, int32_t hp) {
    return launch_dwconv3x3((const half_t*)x, N, H, W, C, (const half_t*)w_rsc, bias, stride, act, (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_stem3x3s2(void* stream, const void* x, int32_t N, int32_t H, int32_t W, const void* wf, const float* bias,
                                 int32_t Kout, int32_t act, void* y, int32_t hp) {
    return launch_stem3x3s2((const half_t*)x, (const half_t*)wf, bias, N, H, W, Kout, act, (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_stem3x3s1(void* stream, const void* x, int32_t N, int32_t H, int32_t W, const void* wf, const float* bias,
                                 int32_t Kout, int32_t act, void* y, int32_t hp) {
    return launch_stem3x3s1((const half_t*)x, (const half_t*)wf, bias, N, H, W, Kout, act, (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_stem3x3s2_dw(void* stream, const void* x, int32_t N, int32_t H, int32_t W, const void* wf, const float* bias,
                                    int32_t act1, const void* wd_rsc, const float* bd, int32_t act2, void* y, int32_t hp) {
    return launch_stem3x3s2_dw((const half_t*)x, (const half_t*)wf, bias, act1, (const half_t*)wd_rsc, bd, act2, N, H, W, (half_t*)y, hp,
                               (hipStream_t)stream);
}
strait_status strait_k_expand_dw(void* stream, const void* x, int32_t N, int32_t H, int32_t W, int32_t Cin, const void* w1,
                                 const float* b1, int32_t Chid, int32_t act1, const void* wd_rsc, const float* bd, int32_t stride,
                                 int32_t act2, void* y, int32_t hp) {
    return launch_expand_dw((const half_t*)x, N, H, W, Cin, (const half_t*)w1, Cin, b1, Chid, act1, (const half_t*)wd_rsc, bd, stride, act2,
                            (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_maxpool3x3s2(void* stream, const void* x, int32_t N, int32_t H, int32_t W, int32_t C, void* y, int32_t hp) {
    return launch_maxpool3x3s2((const half_t*)x, N, H, W, C, (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_stem_pool(void* stream, const void* x, int32_t N, int32_t H, int32_t W, const void* wf, const float* bias,
                                 void* y, int32_t hp) {
    return launch_stem_pool((const half_t*)x, (const half_t*)wf, bias, N, H, W, (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_maxpool2x2s2(void* stream, const void* x, int32_t N, int32_t H, int32_t W, int32_t C, void* y, int32_t hp) {
    return launch_maxpool2x2s2((const half_t*)x, N, H, W, C, (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_vit_tokens(void* stream, const void* patch, const float* cls, const float* pos, int32_t N, int32_t T,
                                  int32_t D, void* z, int32_t hp) {
    return launch_vit_tokens((const half_t*)patch, cls, pos, N, T, D, (half_t*)z, hp, (hipStream_t)stream);
}
strait_status strait_k_global_avgpool(void* stream, const void* x, int32_t N, int32_t HW, int32_t C, void* y, int32_t hp) {
    return launch_global_avgpool((const half_t*)x, N, HW, C, (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_softmax_top1(void* stream, const float* logits, int32_t rows, int32_t n, float* probs, int32_t* top1, int32_t hp) {
    return launch_softmax_top1(logits, rows, n, probs, top1, hp, (hipStream_t)stream);
}
strait_status strait_k_layernorm(void* stream, const void* x, const float* gamma, const float* beta, int32_t rows,
                                 int32_t n, float eps, void* y, int32_t hp) {
    return launch_layernorm((const half_t*)x, gamma, beta, rows, n, eps, (half_t*)y, hp, (hipStream_t)stream);
}
strait_status strait_k_attention(void* stream, const void* qkv, const int32_t* valid_len, int32_t B, int32_t S,
                                 int32_t heads, void* out, int32_t hp) {
    return launch_attention((const half_t*)qkv, valid_len, B, S, heads, (half_t*)out, hp, (hipStream_t)stream);
}
strait_status strait_k_argmax_f16(void* stream, const void* x, int32_t rows, int32_t n, int64_t row_stride, int32_t* top1, int32_t hp) {
    return launch_argmax_f16((const half_t*)x, rows, n, row_stride, top1, hp, (hipStream_t)stream);
}

}  // extern "C"
