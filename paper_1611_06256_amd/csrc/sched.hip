// Queue-driven batching on one GPU (paper Sec. 4.1: prediction queue +
// predictors, training queue + trainers) and the dynamic adjustment of the
// batching knobs (Sec. 4.3), on top of ga3c_predict / ga3c_train_step.
//
// The paper runs predictor and trainer THREADS because each GPU call blocks
// its Python caller.  Here every GPU call only enqueues, so one host thread
// (the caller of ga3c_sched_tick) drains both queues: prediction requests that
// are "immediately available" (Sec. 4.1) go out as one batch on the predict
// stream, trajectories are merged until a minimum batch is reached (Sec. 5.3)
// and go out as one update on the train stream.  The two streams overlap on
// the GPU; the context's parameter snapshots keep a prediction from reading
// half-updated weights.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/ga3c.h"
#include "frame_table.hpp"
#include "sched_error.hpp"

using ga3c::sfail;

namespace {

#define SHIP(expr)                                                                                   \
    do {                                                                                             \
        hipError_t e_ = (expr);                                                                      \
        if (e_ != hipSuccess)                                                                        \
            return sfail(e_ == hipErrorOutOfMemory ? GA3C_ENOMEM : GA3C_EHIP, "%s: %s", #expr,       \
                         hipGetErrorString(e_));                                                     \
    } while (0)

// A batch goes to the GPU as a table of frame pointers and lists of scalars that the host has written into pinned memory:
// where the network's first layer takes frames from a table (frame_table.hpp) its kernels read all of that themselves, other
// networks get their frames put together by a kernel first.  No copy commands either way (a few microseconds of the stream
// each; a round of 256 agents had 24 of them).  Reads of host memory are not cached, so a frame's block asks for its pointer
// once and keeps all of a thread's vectors in flight.
constexpr int GATHER_VPT = 8;        // 16-byte vectors of a frame in flight per thread

__device__ __forceinline__ void copy_frame(const uint4 *__restrict__ s, uint4 *__restrict__ d, int frame_vecs) {
    for (int i0 = threadIdx.x; i0 < frame_vecs; i0 += 256 * GATHER_VPT) {
        uint4 v[GATHER_VPT];
#pragma unroll
        for (int j = 0; j < GATHER_VPT; ++j) v[j] = s[min(i0 + 256 * j, frame_vecs - 1)];
#pragma unroll
        for (int j = 0; j < GATHER_VPT; ++j)
            if (i0 + 256 * j < frame_vecs) d[i0 + 256 * j] = v[j];
    }
}

// Block i: frame i of a prediction batch.
__global__ __launch_bounds__(256) void gather_frames_kernel(const uint4 *const *__restrict__ src_h, uint4 *__restrict__ frames, int frame_vecs) {
    copy_frame(src_h[blockIdx.x], frames + (size_t)blockIdx.x * frame_vecs, frame_vecs);
}

// Block i: experience i of a training batch (frames == nullptr: without its frame); the first n_segments blocks also fetch a
// segment's bootstrap value and start.  *_h: host memory.
struct GatherTrain {
    const uint4 *const *src_h;
    const int32_t *act_h, *seg_h;
    const float *rew_h, *boot_h;
    const uint8_t *done_h;
    uint4 *frames;
    int32_t *act, *seg;
    float *rew, *boot;
    uint8_t *done;
    int frame_vecs, n_segments;
};
__global__ __launch_bounds__(256) void gather_experiences_kernel(const GatherTrain a) {
    const int i = blockIdx.x, t = threadIdx.x;
    if (t == 0) a.act[i] = a.act_h[i];
    if (t == 64) a.rew[i] = a.rew_h[i];
    if (t == 128) a.done[i] = a.done_h[i];
    if (t == 192 && i < a.n_segments) {
        a.boot[i] = a.boot_h[i];
        a.seg[i] = a.seg_h[i];
        if (i == 0) a.seg[a.n_segments] = a.seg_h[a.n_segments];
    }
    if (a.frames) copy_frame(a.src_h[i], a.frames + (size_t)i * a.frame_vecs, a.frame_vecs);
}

}  // namespace

// ------------------------------------------------------------- scheduler ----

namespace {

constexpr int RING = 4;    // batches in flight per stream

struct PredReq { int agent; const uint8_t *frame; float uniform; };
struct Traj {
    int agent;
    int len;                 // experiences in the segment, 1 .. t_max; their actions, rewards and dones lie in the queue's flat lists
    int64_t version;         // updates issued before the policy that chose its first action was read; -1 = not given
    const uint8_t *frames;
    float bootstrap;
};

// First in, first out, in one piece of memory: takes and gives runs of elements without an allocation for each.
template <class T>
struct FlatQueue {
    std::vector<T> v;
    size_t head = 0;
    size_t size() const { return v.size() - head; }
    bool empty() const { return head == v.size(); }
    const T *data() const { return v.data() + head; }
    const T &operator[](size_t i) const { return v[head + i]; }
    // room for n more, or std::bad_alloc with nothing changed; what is pushed into room throws nothing
    void room(size_t n) {
        if (v.capacity() - v.size() < n) v.reserve(std::max(v.size() + n, 2 * v.capacity()));
    }
    void push(const T *p, size_t n) { v.insert(v.end(), p, p + n); }
    void push(const T &x) { v.push_back(x); }
    void pop(size_t n) {
        head += n;
        if (head == v.size()) { v.clear(); head = 0; }
        else if (head > 4096 && head > v.size() / 2) { v.erase(v.begin(), v.begin() + head); head = 0; }
    }
};

struct PredSlot {
    hipEvent_t done = nullptr;
    bool busy = false;
    int n = 0;
    const uint4 **ptrs_h = nullptr;                       // *_h: pinned host memory, which the kernels read and write
    float *unif_h = nullptr;
    int32_t *act_h = nullptr;
    float *val_h = nullptr;
    std::vector<int> agents;
    int64_t version = 0;     // updates issued before this batch
    int seen = 0;            // the first results that have arrived
};

// What a result holds until the kernel's own has arrived: no action is negative, and no arithmetic gives a signalling NaN.
constexpr int32_t NO_ACTION = -1;
constexpr uint32_t NO_VALUE = 0x7fa5a5a5u;

void await_results(PredSlot &p, int n) {
    for (int i = 0; i < n; ++i) p.act_h[i] = NO_ACTION;
    for (int i = 0; i < n; ++i) memcpy(p.val_h + i, &NO_VALUE, sizeof(float));
    p.seen = 0;
}
// Whether all results of the batch lie in the host's memory, which the kernels write.  They do before the event behind the
// batch has completed: that takes the release at the end of the last kernel and a packet of its own (closed loop of 256 agents,
// five predictions and an update: 440 -> 404 us).  The slot is filled again, and the agents' frames are theirs again, from then on:
// the kernels that end a prediction (heads_finish_frame, heads_fwd_kernel) store a frame's value and action once each, behind
// every read of a frame, the table or a uniform number that anything still depends on.
bool results_arrived(PredSlot &p) {
    for (; p.seen < p.n; ++p.seen)
        if (__atomic_load_n(p.act_h + p.seen, __ATOMIC_ACQUIRE) == NO_ACTION ||
            __atomic_load_n((const uint32_t *)p.val_h + p.seen, __ATOMIC_ACQUIRE) == NO_VALUE)
            return false;
    return true;
}

struct TrainSlot {
    hipEvent_t done = nullptr;
    bool busy = false;
    int n_agents = 0;
    const uint4 **ptrs_h = nullptr;
    int32_t *act_h = nullptr, *act_d = nullptr;
    float *rew_h = nullptr, *rew_d = nullptr;
    uint8_t *done_h = nullptr, *done_d = nullptr;
    float *boot_h = nullptr, *boot_d = nullptr;
    int32_t *seg_h = nullptr, *seg_d = nullptr;          // first frame of every segment, and the frame count
};

}  // namespace

struct ga3c_sched {
    ga3c_ctx *ctx;
    ga3c_sched_config cfg;
    ga3c_net_desc desc;
    int max_pred, max_train;
    size_t frame_bytes;
    int predict_cap, train_cap;
    hipStream_t sp, st;
    FlatQueue<PredReq> pq;
    FlatQueue<Traj> tq;
    FlatQueue<int32_t> tq_act;       // of the experiences waiting in tq, segment after segment
    FlatQueue<float> tq_rew;
    FlatQueue<uint8_t> tq_done;
    int64_t tq_frames;       // experiences waiting in tq
    PredSlot ps[RING];
    TrainSlot ts[RING];
    int ps_next, ts_next;
    uint8_t *pred_frames, *train_frames;      // a batch's frames, where the network does not take them from a table: one of each
                                              // will do, since the batches of a kind follow each other on their stream
    FlatQueue<ga3c_prediction> ready;
    ga3c_tuner *tuner;
    ga3c_sched_stats stats;
    int64_t window_ticks, window_frames;
    std::chrono::steady_clock::time_point window_start;
};

namespace {

// Coherent: the host reads results while the kernels that store them run (results_arrived), and kernels read lists that the
// host has just written; what the default is can be changed from outside (HIP_HOST_COHERENT).
template <class T>
int pinned(T **p, size_t n) {
    SHIP(hipHostMalloc((void **)p, sizeof(T) * std::max<size_t>(n, 1), hipHostMallocCoherent));
    return GA3C_OK;
}
template <class T>
int device(T **p, size_t n) {
    SHIP(hipMalloc((void **)p, sizeof(T) * std::max<size_t>(n, 1)));
    return GA3C_OK;
}
// A queue that cannot grow is an error code at the C boundary.
#define NO_MEMORY(what) catch (const std::bad_alloc &) { return sfail(GA3C_ENOMEM, what ": out of memory"); }
#define STRY(expr) do { int rc_ = (expr); if (rc_ != GA3C_OK) return rc_; } while (0)

int alloc_slots(ga3c_sched *s) {
    const int maxN = s->max_train;      // a segment has at least one frame
    // also for a network that takes a table: ga3c_use_generic_kernels may come at any time, and a tick allocates nothing
    STRY(device(&s->pred_frames, (size_t)s->max_pred * s->frame_bytes));
    STRY(device(&s->train_frames, (size_t)s->max_train * s->frame_bytes));
    for (int i = 0; i < RING; ++i) {
        PredSlot &p = s->ps[i];
        SHIP(hipEventCreateWithFlags(&p.done, hipEventDisableTiming));
        STRY(pinned(&p.ptrs_h, s->max_pred));
        STRY(pinned(&p.unif_h, s->max_pred));
        STRY(pinned(&p.act_h, s->max_pred)); STRY(pinned(&p.val_h, s->max_pred));
        try { p.agents.reserve(s->max_pred); } NO_MEMORY("ga3c_sched_create")
        TrainSlot &t = s->ts[i];
        SHIP(hipEventCreateWithFlags(&t.done, hipEventDisableTiming));
        STRY(pinned(&t.ptrs_h, maxN));
        STRY(pinned(&t.act_h, s->max_train)); STRY(device(&t.act_d, s->max_train));
        STRY(pinned(&t.rew_h, s->max_train)); STRY(device(&t.rew_d, s->max_train));
        STRY(pinned(&t.done_h, s->max_train)); STRY(device(&t.done_d, s->max_train));
        STRY(pinned(&t.boot_h, maxN)); STRY(device(&t.boot_d, maxN));
        STRY(pinned(&t.seg_h, maxN + 1)); STRY(device(&t.seg_d, maxN + 1));
    }
    return GA3C_OK;
}

// Moves the results of finished prediction batches to the ready list.
int harvest(ga3c_sched *s, bool wait) {
    for (int k = 0; k < RING; ++k) {
        PredSlot &p = s->ps[(s->ps_next + k) % RING];        // oldest first
        if (!p.busy) continue;
        if (wait) SHIP(hipEventSynchronize(p.done));
        else if (!results_arrived(p)) {
            const hipError_t q = hipEventQuery(p.done);
            if (q == hipErrorNotReady) break;                // a later one that is over by now waits for this one
            if (q != hipSuccess) return sfail(GA3C_EHIP, "hipEventQuery: %s", hipGetErrorString(q));
        }
        try { s->ready.room(p.n); } NO_MEMORY("ga3c_sched: results")
        for (int i = 0; i < p.n; ++i)
            s->ready.push(ga3c_prediction{p.agents[i], p.act_h[i], p.val_h[i], (int32_t)p.version});
        p.busy = false;
    }
    for (int k = 0; k < RING; ++k) {
        TrainSlot &t = s->ts[k];
        if (!t.busy) continue;
        if (wait) SHIP(hipEventSynchronize(t.done));
        else if (hipEventQuery(t.done) != hipSuccess) continue;
        t.busy = false;
    }
    return GA3C_OK;
}

// What a batch that could not be enqueued whole has left on its stream reads the slot's lists and writes its results: it has to be
// over before the slot is filled again.  Returns the batch's code.
int abandon(hipStream_t stream, int rc) {
    (void)hipStreamSynchronize(stream);
    return rc;
}

int enqueue_predict(ga3c_sched *s, PredSlot &p, int n) {
    int rc;
    if (ga3c::takes_frame_table(s->ctx))
        rc = ga3c::predict_from_table(s->ctx, (const uint8_t *const *)p.ptrs_h, n, p.unif_h, p.val_h, p.act_h, s->sp);
    else {
        hipLaunchKernelGGL(gather_frames_kernel, dim3(n), dim3(256), 0, s->sp, p.ptrs_h, (uint4 *)s->pred_frames, (int)(s->frame_bytes / 16));
        SHIP(hipGetLastError());
        rc = ga3c_predict(s->ctx, s->pred_frames, n, p.unif_h, nullptr, p.val_h, nullptr, p.act_h, s->sp);
    }
    if (rc != GA3C_OK) return sfail(GA3C_EHIP, "ga3c_predict: %s", ga3c_last_error());
    SHIP(hipEventRecord(p.done, s->sp));
    return GA3C_OK;
}

int issue_predict(ga3c_sched *s, int *count) {
    *count = 0;
    if (s->pq.empty()) return GA3C_OK;
    if ((int)s->pq.size() < s->predict_cap) {
        // Fewer requests than a full batch: they go out at once only if no earlier batch is still in flight;
        // otherwise they wait for it, and what arrives meanwhile joins them.  (A single predictor of Sec. 4.1 behaves
        // like this: it is busy with its batch.  Full batches are issued back to back, up to RING of them, like
        // several predictors.)  Under light load this makes batches as large as the GPU's own pace allows.
        STRY(harvest(s, false));
        for (int k = 0; k < RING; ++k)
            if (s->ps[k].busy) return GA3C_OK;
    }
    PredSlot &p = s->ps[s->ps_next];
    if (p.busy) {                                   // ring full: wait for the oldest batch
        SHIP(hipEventSynchronize(p.done));
        STRY(harvest(s, false));
    }
    // the requests leave the queue only when the whole batch has been enqueued: a failing GPU call loses none
    const int n = (int)std::min<size_t>(s->pq.size(), (size_t)s->predict_cap);
    p.agents.resize(n);
    for (int i = 0; i < n; ++i) {
        const PredReq &r = s->pq[i];
        p.agents[i] = r.agent; p.ptrs_h[i] = (const uint4 *)r.frame; p.unif_h[i] = r.uniform;
    }
    await_results(p, n);
    if (const int rc = enqueue_predict(s, p, n); rc != GA3C_OK) return abandon(s->sp, rc);
    s->pq.pop(n);
    p.busy = true; p.n = n;
    p.version = s->stats.train_batches;      // the call above reads the parameters that this many updates produced
    s->ps_next = (s->ps_next + 1) % RING;
    s->stats.predictions += n; s->stats.predict_batches += 1;
    *count = n;
    return GA3C_OK;
}

// n segments of B frames in all, the lists of which lie in the slot.
int enqueue_train(ga3c_sched *s, TrainSlot &t, int n, int B, bool equal) {
    const int T = s->cfg.t_max;
    const bool table = ga3c::takes_frame_table(s->ctx);
    int rc;
    if (table && equal) {        // every list is read where the host wrote it
        rc = ga3c::train_from_table(s->ctx, (const uint8_t *const *)t.ptrs_h, t.act_h, t.rew_h, t.done_h, t.boot_h, nullptr, n, T, B, &s->cfg.hp, s->st);
    } else {
        const GatherTrain ga{t.ptrs_h, t.act_h, t.seg_h, t.rew_h, t.boot_h, t.done_h, table ? nullptr : (uint4 *)s->train_frames, t.act_d, t.seg_d,
                             t.rew_d, t.boot_d, t.done_d, (int)(s->frame_bytes / 16), n};
        hipLaunchKernelGGL(gather_experiences_kernel, dim3(B), dim3(256), 0, s->st, ga);
        SHIP(hipGetLastError());
        rc = table   ? ga3c::train_from_table(s->ctx, (const uint8_t *const *)t.ptrs_h, t.act_d, t.rew_d, t.done_d, t.boot_d, t.seg_d, n, 1, B,
                                              &s->cfg.hp, s->st)
             : equal ? ga3c_train_step(s->ctx, s->train_frames, t.act_d, t.rew_d, t.done_d, t.boot_d, n, T, &s->cfg.hp, nullptr, s->st)
                     : ga3c_train_step_ragged(s->ctx, s->train_frames, t.act_d, t.rew_d, t.done_d, t.seg_d, t.boot_d, n, B, &s->cfg.hp, nullptr, s->st);
    }
    if (rc != GA3C_OK) return sfail(GA3C_EHIP, "ga3c_train_step: %s", ga3c_last_error());
    SHIP(hipEventRecord(t.done, s->st));
    return GA3C_OK;
}

int issue_train(ga3c_sched *s, int *count) {
    *count = 0;
    const int T = s->cfg.t_max;
    // merge until the minimum batch is there (Sec. 5.3).  With the adjustment on, its training knob is the batch size
    // itself: an update waits for train_cap frames and takes at most as many, so the knob decides how large the
    // updates are whatever the pace at which segments arrive
    const int need = s->tuner ? std::max(s->cfg.train_min, s->train_cap) : s->cfg.train_min;
    if (s->tq.empty() || s->tq_frames < need) return GA3C_OK;
    TrainSlot &t = s->ts[s->ts_next];
    if (t.busy) {
        SHIP(hipEventSynchronize(t.done));
        t.busy = false;
    }
    // whole segments, oldest first, while they fit the cap (the first one always goes); they leave the queue, and
    // enter the statistics, only when the update has been enqueued: a failing GPU call loses none
    int n = 0, B = 0;
    bool equal = true;
    while ((size_t)n < s->tq.size() && (n == 0 || B + s->tq[n].len <= s->train_cap)) {
        const Traj &tr = s->tq[n];
        const int L = tr.len;
        for (int k = 0; k < L; ++k) t.ptrs_h[B + k] = (const uint4 *)(tr.frames + (size_t)k * s->frame_bytes);
        t.boot_h[n] = tr.bootstrap;
        t.seg_h[n] = B;
        if (L != T) equal = false;
        B += L; n += 1;
    }
    t.seg_h[n] = B;
    memcpy(t.act_h, s->tq_act.data(), sizeof(int32_t) * B);
    memcpy(t.rew_h, s->tq_rew.data(), sizeof(float) * B);
    memcpy(t.done_h, s->tq_done.data(), B);
    if (const int rc = enqueue_train(s, t, n, B, equal); rc != GA3C_OK) return abandon(s->st, rc);
    const int64_t now = s->stats.train_batches;       // updates issued before this one = the version it starts from
    for (int i = 0; i < n; ++i) {
        const Traj &tr = s->tq[i];
        if (tr.len != T) s->stats.short_segments += 1;
        if (tr.version >= 0) {
            const int64_t lag = now - tr.version;
            s->stats.lag_sum += lag; s->stats.lag_count += 1;
            s->stats.lag_max = std::max(s->stats.lag_max, lag);
        }
        s->tq_frames -= tr.len;
    }
    s->tq.pop(n); s->tq_act.pop(B); s->tq_rew.pop(B); s->tq_done.pop(B);
    t.busy = true; t.n_agents = n;
    s->ts_next = (s->ts_next + 1) % RING;
    s->stats.trained_frames += (int64_t)B; s->stats.train_batches += 1;
    *count = B;
    return GA3C_OK;
}

}  // namespace

extern "C" int ga3c_sched_create(ga3c_ctx *ctx, const ga3c_sched_config *cfg, ga3c_sched **out) {
    if (out) *out = nullptr;
    if (!ctx || !cfg || !out) return sfail(GA3C_EINVAL, "ga3c_sched_create: null argument");
    ga3c_net_desc d;
    int mp, mt;
    if (ga3c_get_desc(ctx, &d, &mp, &mt) != GA3C_OK) return sfail(GA3C_EINVAL, "ga3c_sched_create: bad context");
    const size_t fb = (size_t)d.in_c * d.in_h * d.in_w;
    if (fb % 16 != 0) return sfail(GA3C_EINVAL, "ga3c_sched_create: frame size must be a multiple of 16 bytes");
    if (cfg->t_max < 1 || cfg->predict_cap < 1 || cfg->predict_cap > mp || cfg->train_min < 1 ||
        cfg->train_cap < cfg->t_max || cfg->train_cap > mt || cfg->train_min > cfg->train_cap)
        return sfail(GA3C_EINVAL, "ga3c_sched_create: caps outside the context's capacity (predict %d, train %d)", mp, mt);
    if (cfg->adjust_period > 0 &&
        (cfg->predict_cap_lo < 1 || cfg->predict_cap_hi > mp || cfg->predict_cap_lo > cfg->predict_cap ||
         cfg->predict_cap_hi < cfg->predict_cap || cfg->train_cap_lo < cfg->train_min || cfg->train_cap_hi > mt ||
         cfg->train_cap_lo > cfg->train_cap || cfg->train_cap_hi < cfg->train_cap || cfg->train_cap_step < 1))
        return sfail(GA3C_EINVAL, "ga3c_sched_create: adjustment bounds must contain the initial caps and fit the context");
    ga3c_sched *s = new (std::nothrow) ga3c_sched();
    if (!s) return sfail(GA3C_ENOMEM, "ga3c_sched_create: out of memory");
    s->ctx = ctx; s->cfg = *cfg; s->desc = d; s->max_pred = mp; s->max_train = mt; s->frame_bytes = fb;
    s->predict_cap = cfg->predict_cap; s->train_cap = cfg->train_cap;
    s->sp = s->st = nullptr; s->ps_next = s->ts_next = 0; s->pred_frames = s->train_frames = nullptr; s->tuner = nullptr; s->tq_frames = 0;
    memset(&s->stats, 0, sizeof(s->stats));
    s->stats.predict_cap = s->predict_cap; s->stats.train_cap = s->train_cap;
    s->window_ticks = s->window_frames = 0;
    int rc = GA3C_OK;
    // default priority for both streams
    if (hipStreamCreateWithFlags(&s->sp, hipStreamNonBlocking) != hipSuccess ||
        hipStreamCreateWithFlags(&s->st, hipStreamNonBlocking) != hipSuccess)
        rc = sfail(GA3C_EHIP, "ga3c_sched_create: hipStreamCreate failed");
    if (rc == GA3C_OK) rc = alloc_slots(s);
    if (rc == GA3C_OK && cfg->adjust_period > 0)
        rc = ga3c_tuner_create(cfg->predict_cap_lo, cfg->predict_cap_hi, cfg->predict_cap, cfg->train_cap_lo,
                               cfg->train_cap_hi, cfg->train_cap_step, cfg->train_cap, cfg->seed, &s->tuner);
    if (rc == GA3C_OK && s->tuner && cfg->adjust_margin > 0.f) rc = ga3c_tuner_set_margin(s->tuner, cfg->adjust_margin);
    if (rc != GA3C_OK) {
        char keep[512];
        snprintf(keep, sizeof(keep), "%s", ga3c::sched_error_text());
        ga3c_sched_destroy(s);
        sfail(rc, "%s", keep);
        return rc;
    }
    s->window_start = std::chrono::steady_clock::now();
    *out = s;
    return GA3C_OK;
}

extern "C" int ga3c_sched_destroy(ga3c_sched *s) {
    if (!s) return GA3C_OK;
    if (s->sp) (void)hipStreamSynchronize(s->sp);
    if (s->st) (void)hipStreamSynchronize(s->st);
    for (int i = 0; i < RING; ++i) {
        PredSlot &p = s->ps[i];
        if (p.done) (void)hipEventDestroy(p.done);
        (void)hipHostFree(p.ptrs_h); (void)hipHostFree(p.unif_h);
        (void)hipHostFree(p.act_h); (void)hipHostFree(p.val_h);
        TrainSlot &t = s->ts[i];
        if (t.done) (void)hipEventDestroy(t.done);
        (void)hipHostFree(t.ptrs_h);
        (void)hipHostFree(t.act_h); (void)hipFree(t.act_d); (void)hipHostFree(t.rew_h); (void)hipFree(t.rew_d);
        (void)hipHostFree(t.done_h); (void)hipFree(t.done_d); (void)hipHostFree(t.boot_h); (void)hipFree(t.boot_d);
        (void)hipHostFree(t.seg_h); (void)hipFree(t.seg_d);
    }
    (void)hipFree(s->pred_frames); (void)hipFree(s->train_frames);
    if (s->sp) (void)hipStreamDestroy(s->sp);
    if (s->st) (void)hipStreamDestroy(s->st);
    ga3c_tuner_destroy(s->tuner);
    delete s;
    return GA3C_OK;
}

extern "C" int ga3c_sched_submit_predict(ga3c_sched *s, int agent, const uint8_t *frame_dev, float uniform) {
    if (!s || !frame_dev) return sfail(GA3C_EINVAL, "ga3c_sched_submit_predict: null argument");
    if (((uintptr_t)frame_dev) & 15) return sfail(GA3C_EINVAL, "ga3c_sched_submit_predict: frame must be 16-byte aligned");
    try { s->pq.room(1); } NO_MEMORY("ga3c_sched_submit_predict")
    s->pq.push(PredReq{agent, frame_dev, uniform});
    return GA3C_OK;
}

extern "C" int ga3c_sched_submit_segment(ga3c_sched *s, int agent, const uint8_t *frames_dev, int len,
                                         const int32_t *actions, const float *rewards, const uint8_t *dones,
                                         float bootstrap, int64_t policy_version) {
    if (!s || !frames_dev || !actions || !rewards || !dones)
        return sfail(GA3C_EINVAL, "ga3c_sched_submit_segment: null argument");
    if (((uintptr_t)frames_dev) & 15)
        return sfail(GA3C_EINVAL, "ga3c_sched_submit_segment: frames must be 16-byte aligned");
    if (len < 1 || len > s->cfg.t_max)
        return sfail(GA3C_EINVAL, "ga3c_sched_submit_segment: length %d outside 1..t_max = %d", len, s->cfg.t_max);
    for (int i = 0; i < len; ++i)
        if (actions[i] < 0 || actions[i] >= s->desc.n_actions)
            return sfail(GA3C_EINVAL, "ga3c_sched_submit_segment: action %d out of range", (int)actions[i]);
    Traj tr;
    tr.agent = agent; tr.len = len; tr.version = policy_version < 0 ? -1 : policy_version;
    tr.frames = frames_dev; tr.bootstrap = bootstrap;
    try { s->tq_act.room(len); s->tq_rew.room(len); s->tq_done.room(len); s->tq.room(1); } NO_MEMORY("ga3c_sched_submit_segment")
    s->tq_act.push(actions, len);
    s->tq_rew.push(rewards, len);
    s->tq_done.push(dones, len);
    s->tq.push(tr);
    s->tq_frames += len;
    return GA3C_OK;
}

extern "C" int ga3c_sched_submit_trajectory(ga3c_sched *s, int agent, const uint8_t *frames_dev, const int32_t *actions,
                                            const float *rewards, const uint8_t *dones, float bootstrap) {
    if (!s) return sfail(GA3C_EINVAL, "ga3c_sched_submit_trajectory: null scheduler");
    return ga3c_sched_submit_segment(s, agent, frames_dev, s->cfg.t_max, actions, rewards, dones, bootstrap, -1);
}

extern "C" int ga3c_sched_submit_predict_many(ga3c_sched *s, int n, const int32_t *agents,
                                              const uint8_t *const *frames_dev, const float *uniforms) {
    if (!s || n < 0 || (n > 0 && (!agents || !frames_dev || !uniforms)))
        return sfail(GA3C_EINVAL, "ga3c_sched_submit_predict_many: bad argument");
    for (int i = 0; i < n; ++i)
        if (!frames_dev[i] || (((uintptr_t)frames_dev[i]) & 15))
            return sfail(GA3C_EINVAL, "ga3c_sched_submit_predict_many: frame %d is null or not 16-byte aligned", i);
    try { s->pq.room(n); } NO_MEMORY("ga3c_sched_submit_predict_many")
    for (int i = 0; i < n; ++i) s->pq.push(PredReq{agents[i], frames_dev[i], uniforms[i]});
    return GA3C_OK;
}

extern "C" int ga3c_sched_submit_trajectory_many(ga3c_sched *s, int n, const int32_t *agents,
                                                 const uint8_t *const *frames_dev, const int32_t *actions,
                                                 const float *rewards, const uint8_t *dones, const float *bootstrap) {
    if (!s || n < 0 || (n > 0 && (!agents || !frames_dev || !actions || !rewards || !dones || !bootstrap)))
        return sfail(GA3C_EINVAL, "ga3c_sched_submit_trajectory_many: bad argument");
    const int T = s->cfg.t_max;
    for (int i = 0; i < n; ++i) {
        const int rc = ga3c_sched_submit_trajectory(s, agents[i], frames_dev[i], actions + (size_t)i * T,
                                                    rewards + (size_t)i * T, dones + (size_t)i * T, bootstrap[i]);
        if (rc != GA3C_OK) return rc;
    }
    return GA3C_OK;
}

extern "C" int ga3c_sched_submit_segment_many(ga3c_sched *s, int n, const int32_t *agents,
                                              const uint8_t *const *frames_dev, const int32_t *lens,
                                              const int32_t *actions, const float *rewards, const uint8_t *dones,
                                              const float *bootstrap, const int64_t *policy_versions) {
    if (!s || n < 0 || (n > 0 && (!agents || !frames_dev || !lens || !actions || !rewards || !dones || !bootstrap)))
        return sfail(GA3C_EINVAL, "ga3c_sched_submit_segment_many: bad argument");
    const int T = s->cfg.t_max;
    for (int i = 0; i < n; ++i) {
        const int rc = ga3c_sched_submit_segment(s, agents[i], frames_dev[i], lens[i], actions + (size_t)i * T,
                                                 rewards + (size_t)i * T, dones + (size_t)i * T, bootstrap[i],
                                                 policy_versions ? policy_versions[i] : -1);
        if (rc != GA3C_OK) return rc;
    }
    return GA3C_OK;
}

extern "C" int ga3c_sched_tick(ga3c_sched *s, int *predicted, int *trained) {
    if (!s) return sfail(GA3C_EINVAL, "ga3c_sched_tick: null scheduler");
    int np = 0, nt = 0;
    s->stats.ticks += 1;
    s->stats.sum_predict_queue += (int64_t)s->pq.size();
    s->stats.sum_train_queue += (int64_t)s->tq.size();
    STRY(issue_predict(s, &np));
    STRY(issue_train(s, &nt));
    STRY(harvest(s, false));
    if (predicted) *predicted = np;
    if (trained) *trained = nt;
    if (s->tuner) {
        s->window_ticks += 1; s->window_frames += nt;
        if (s->window_ticks >= s->cfg.adjust_period) {
            // throughput of the window that just ended: finish its GPU work, then read the clock
            SHIP(hipStreamSynchronize(s->st));
            SHIP(hipStreamSynchronize(s->sp));
            const auto now = std::chrono::steady_clock::now();
            const double sec = std::chrono::duration<double>(now - s->window_start).count();
            const double thr = sec > 0 ? (double)s->window_frames / sec : 0.0;
            ga3c_tuner_report(s->tuner, thr, &s->predict_cap, &s->train_cap);
            s->stats.last_window_frames_per_s = thr;
            s->stats.predict_cap = s->predict_cap; s->stats.train_cap = s->train_cap;
            ga3c_tuner_state(s->tuner, nullptr, nullptr, &s->stats.trials_accepted, &s->stats.trials_rejected);
            ga3c_tuner_progress(s->tuner, &s->stats.windows, &s->stats.last_change_window);
            s->window_ticks = s->window_frames = 0;
            s->window_start = std::chrono::steady_clock::now();
        }
    }
    return GA3C_OK;
}

extern "C" int ga3c_sched_poll(ga3c_sched *s, ga3c_prediction *out, int cap) {
    if (!s || (!out && cap > 0) || cap < 0) return sfail(GA3C_EINVAL, "ga3c_sched_poll: bad argument");
    STRY(harvest(s, false));
    const int n = (int)std::min<size_t>(s->ready.size(), (size_t)cap);
    if (n > 0) memcpy(out, s->ready.data(), sizeof(ga3c_prediction) * n);
    s->ready.pop(n);
    return n;
}

extern "C" int ga3c_sched_drain(ga3c_sched *s) {
    if (!s) return sfail(GA3C_EINVAL, "ga3c_sched_drain: null scheduler");
    SHIP(hipStreamSynchronize(s->sp));
    SHIP(hipStreamSynchronize(s->st));
    return harvest(s, true);
}

extern "C" int ga3c_sched_get_stats(const ga3c_sched *s, ga3c_sched_stats *out) {
    if (!s || !out) return sfail(GA3C_EINVAL, "ga3c_sched_get_stats: null argument");
    *out = s->stats;
    out->predict_queue = (int64_t)s->pq.size();
    out->train_queue = (int64_t)s->tq.size();
    return GA3C_OK;
}

