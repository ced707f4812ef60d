// The library's host code (csrc/ga3c.hip, sched.hip, tuner.cpp) on a stand-in for the HIP runtime that runs nothing and keeps
// account: for every launch, which earlier launches it is ordered behind (stream order, events, host waits), for every handle
// whether the call that uses it was given it, and what is allocated when.  No GPU.  Built and run by tests/test_host_path_cpu.py
// with the name of a check as its argument.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <set>
#include <string>
#include <vector>

#include "../include/ga3c.h"

static int problems = 0;
#define PROBLEM(...) do { if (++problems <= 20) { printf("problem: " __VA_ARGS__); printf("\n"); } } while (0)

static int memory_left = -1;                          // allocations until one fails; -1: none does
static int launches_left = -1, records_left = -1;     // launches, and event records, until one fails
static bool launch_failed = false;
static bool fails(int &left) { return left >= 0 && left-- == 0; }
void *operator new(size_t n) {
    if (memory_left >= 0 && memory_left-- == 0) throw std::bad_alloc();
    if (void *p = malloc(n ? n : 1)) return p;
    abort();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

// ------------------------------------------------------------------ the stand-in runtime --

typedef std::vector<bool> Seen;                       // launches that something is ordered behind
static void join(Seen &a, const Seen &b) {
    if (a.size() < b.size()) a.resize(b.size());
    for (size_t i = 0; i < b.size(); ++i) if (b[i]) a[i] = true;
}
struct Op { std::string name; Seen before; const void *to = nullptr, *from = nullptr; };      // to, from: of kernels that copy or update
struct Stream { bool alive = true, capturing = false; Seen seen; };
struct Event { Seen seen; bool alive = true; };
static std::vector<Op> ops;
static std::map<hipStream_t, Stream> streams;
static std::map<hipEvent_t, Event> events;
static std::map<void *, size_t> device_memory;
static std::map<const void *, std::string> kernels;
static std::set<hipStream_t> given;                   // handles that the running call may use
static Seen host;                                     // launches known to be over
static bool in_call = false;                          // inside a call that only enqueues
static int allocations = 0, records = 0;
static size_t device_bytes = 0, last_bytes = 0;      // device memory held, and asked for last

static Stream *use(hipStream_t s, const char *what) {
    if (in_call && !given.count(s)) PROBLEM("%s on a stream that the call was not given", what);
    Stream &t = streams[s];
    if (!t.alive) PROBLEM("%s on a stream that is gone", what);
    return &t;
}
static void put(hipStream_t s, const std::string &name, const void *to = nullptr, const void *from = nullptr) {
    Stream *t = use(s, name.c_str());
    join(t->seen, host);
    ops.push_back(Op{name, t->seen, to, from});
    t->seen.resize(ops.size());
    t->seen.back() = true;
}
static void host_wait(const char *what, const Seen &seen) {
    if (in_call) PROBLEM("%s inside a call that only enqueues", what);
    join(host, seen);
}
static Seen everything() { return Seen(ops.size(), true); }

extern "C" {
struct Fake { int x; };
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) { cfg_grid = g; cfg_block = b; cfg_lds = l; cfg_stream = s; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s) { *g = cfg_grid; *b = cfg_block; *l = cfg_lds; *s = cfg_stream; return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host_fn, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { kernels[host_fn] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

static void launched(const void *f, void **args, hipStream_t s) {
    const std::string &name = kernels[f];
    const bool rms = name.find("rmsprop_kernel") != std::string::npos, fill = name.find("fill_kernel") != std::string::npos, copy = name.find("copy_kernel") != std::string::npos;
    const void *a = rms || fill || copy ? *(void **)args[0] : nullptr, *b = rms || copy ? *(void **)args[1] : nullptr;
    put(s, name, rms ? b : a, rms ? a : b);
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t s) {
    if (fails(launches_left)) { launch_failed = true; return hipErrorUnknown; }
    launched(f, args, s);
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t s, hipEvent_t, hipEvent_t stop, int) {
    launched(f, args, s);
    if (streams[s].capturing) PROBLEM("a launch with events of its own on a stream that is being captured");
    if (stop) events[stop].seen = streams[s].seen;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *from, size_t, hipMemcpyKind, hipStream_t s) { put(s, "memcpy", to, from); return hipSuccess; }
hipError_t hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, hipMemcpyKind, hipStream_t s) { put(s, "memcpy"); return hipSuccess; }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { host_wait("hipMemcpy", Seen()); return hipSuccess; }
hipError_t hipMemset(void *, int, size_t) { if (in_call) PROBLEM("hipMemset inside a call that only enqueues"); return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { host_wait("hipDeviceSynchronize", everything()); return hipSuccess; }

static hipError_t new_event(hipEvent_t *e) { *e = (hipEvent_t)new Fake(); events[*e] = Event(); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return new_event(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return new_event(e); }
hipError_t hipEventDestroy(hipEvent_t e) { events[e].alive = false; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    if (fails(records_left)) return hipErrorUnknown;
    ++records;
    events[e].seen = use(s, "hipEventRecord")->seen;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { join(use(s, "hipStreamWaitEvent")->seen, events[e].seen); return hipSuccess; }
static int queries_left = -1;                         // event queries until one finds its event not completed
hipError_t hipEventQuery(hipEvent_t e) {
    if (fails(queries_left)) return hipErrorNotReady;
    join(host, events[e].seen);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { join(host, events[e].seen); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)new Fake(); streams[*s] = Stream(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { streams[s].alive = false; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { host_wait("hipStreamSynchronize", streams[s].seen); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) {
    *st = use(s, "hipStreamIsCapturing")->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}

static hipError_t take(void **p, size_t n) {
    ++allocations;
    if (in_call) PROBLEM("%zu bytes allocated inside a call that only enqueues", n);
    *p = malloc(n < 4096 ? n : 4096);                 // device memory is never touched here
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { take(p, n); device_memory[*p] = n; device_bytes += n; last_bytes = n; return hipSuccess; }
hipError_t hipFree(void *p) { if (p) { device_bytes -= device_memory[p]; device_memory.erase(p); free(p); } return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags) {
    ++allocations;
    if (in_call) PROBLEM("hipHostMalloc inside a call that only enqueues");
    if (!(flags & hipHostMallocCoherent)) PROBLEM("host memory that is not asked for as coherent");      // results are read while kernels run
    *p = calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipGetLastError(void) { const hipError_t e = launch_failed ? hipErrorUnknown : hipSuccess; launch_failed = false; return e; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char at[256]; *p = at; return hipSuccess; }
}

// ------------------------------------------------------------------ the checks ------------

static hipStream_t new_stream() { hipStream_t s; (void)hipStreamCreateWithFlags(&s, 0); return s; }
static uint8_t *address(size_t i) { return (uint8_t *)(uintptr_t)(4096 + 16 * i); }      // never read

static ga3c_net_desc net_desc(const char *net) {
    ga3c_net_desc d;
    memset(&d, 0, sizeof(d));
    d.in_c = 4; d.in_h = d.in_w = 84; d.n_actions = 6;
    auto conv = [&](int oc, int k, int stride) { d.conv[d.n_conv].oc = oc; d.conv[d.n_conv].k = k; d.conv[d.n_conv++].stride = stride; };
    if (!strcmp(net, "small")) { conv(16, 8, 4); conv(32, 4, 2); d.fc_units = 256; }
    else if (!strcmp(net, "large")) { conv(32, 8, 4); conv(64, 4, 2); conv(64, 3, 1); d.fc_units = 512; }
    else { conv(32, 8, atoi(net + 5)); conv(32, 4, 2); conv(64, 4, 2); d.fc_units = 256; }
    return d;
}

// A context, and who reads and writes its parameter copies when.
struct Program {
    ga3c_ctx *ctx = nullptr;
    const void *published = nullptr;                  // the copy that was written last
    std::map<const void *, std::vector<int>> writer, readers;      // launches that the next reader / the next writer has to come after
    // calls of a kind (0 predictions, 1 updates and what else writes the parameters) on several streams are in order among
    // themselves: the program's own events see to that
    hipStream_t last[2] = {nullptr, nullptr};
    hipEvent_t own[2] = {nullptr, nullptr};
    bool gets_ordered = true;                         // read-outs on the updates' stream too, when the updates move to another
    ga3c_hparams hp = {0.99f, 0.01f, 1.f, 0.f, 1e-4f, 0.99f, 0.1f, 40.f};

    explicit Program(const char *net, int pred = 64, int train = 160) {
        const ga3c_net_desc d = net_desc(net);
        if (ga3c_create(&d, pred, train, &ctx) != GA3C_OK) PROBLEM("create: %s", ga3c_last_error());
    }
    ~Program() { ga3c_destroy(ctx); }

    static void behind(int op, const std::vector<int> &must, const char *what) {
        for (int m : must)
            if (!(m < (int)ops[op].before.size() && ops[op].before[m])) { PROBLEM("%s (%s) is not ordered behind %s", what, ops[op].name.c_str(), ops[m].name.c_str()); return; }
    }
    void before_own(int kind, hipStream_t s) { if (own[kind] && last[kind] != s) (void)hipStreamWaitEvent(s, own[kind], 0); }
    void after_own(int kind, hipStream_t s) {
        if (!own[kind]) new_event(&own[kind]);
        events[own[kind]].seen = streams[s].seen;
        last[kind] = s;
    }
    template <class F>
    int call(hipStream_t s, F f) {
        const int first = (int)ops.size();
        given = {s}; in_call = true;
        if (f() != GA3C_OK) PROBLEM("a call failed: %s", ga3c_last_error());
        in_call = false;
        if (first == (int)ops.size()) PROBLEM("a call launched nothing");
        return first;
    }
    // launch `op` overwrote copy `to` for good
    void wrote(int op, const void *to, const char *what) {
        behind(op, writer[to], what); behind(op, readers[to], what);
        writer[to] = {(int)ops.size() - 1}; readers[to].clear();
        published = to;
    }
    void init(hipStream_t s, bool set = false) {
        before_own(1, s);
        const int first = call(s, [&] { return set ? ga3c_params_set(ctx, 0, (const float *)address(1), ga3c_params_count(ctx), s) : ga3c_params_init(ctx, 1, s); });
        behind(first, writer[published], "parameters written");
        wrote(first, ops[first].to, "parameters written");
        after_own(1, s);
    }
    void get(hipStream_t s) {
        const int first = call(s, [&] { return ga3c_params_get(ctx, 0, (float *)address(1), ga3c_params_count(ctx), s); });
        if (ops[first].from != published) PROBLEM("a read-out of another copy than the published one");
        behind(first, writer[published], "a read-out");
        readers[published].push_back(first);
        if (gets_ordered && own[1] && s == last[1]) after_own(1, s);
    }
    void predict(hipStream_t s, int B) {
        before_own(0, s);
        const int first = call(s, [&] { return ga3c_predict(ctx, address(0), B, nullptr, nullptr, (float *)address(1), nullptr, nullptr, s); });
        behind(first, writer[published], "a prediction");
        readers[published].push_back((int)ops.size() - 1);
        after_own(0, s);
    }
    void train(hipStream_t s, int N) {
        before_own(1, s);
        const int first = call(s, [&] { return ga3c_train_step(ctx, address(0), (const int32_t *)address(1), (const float *)address(2), address(3), nullptr, N, 5, &hp, nullptr, s); });
        behind(first, writer[published], "an update");
        int rms = -1;
        for (int i = first; i < (int)ops.size(); ++i) if (ops[i].name.find("rmsprop") != std::string::npos) rms = i;
        if (rms < 0) { PROBLEM("an update without rmsprop"); return; }
        if (ops[rms].from != published) PROBLEM("an update of another copy than the published one");
        readers[published].push_back(rms);
        if (ops[rms].to == published) readers[published].pop_back();
        wrote(rms, ops[rms].to, "the new parameters");
        after_own(1, s);
    }
    void over(hipStream_t s) { (void)hipStreamSynchronize(s); }
};

static unsigned rng_state = 12345;
static int any(int n) { rng_state = rng_state * 1664525u + 1013904223u; return (int)((rng_state >> 16) % (unsigned)n); }

// Calls that wander over streams, also over streams that go away and whose handle comes back as another stream's.
static void streams_check() {
    for (const char *net : {"small", "large", "paper3"}) {
        {   // the stream of the first calls is gone when the second one appears
            Program p(net);
            hipStream_t a = new_stream(), b = new_stream();
            p.init(a); p.predict(a, 64); p.train(a, 8); p.predict(a, 3);
            (void)hipStreamDestroy(a);
            p.train(b, 8); p.train(b, 8);
        }
        {   // its handle stands for another stream by then
            Program p(net);
            hipStream_t a = new_stream(), b = new_stream();
            p.init(a); p.predict(a, 64); p.predict(a, 3);
            streams[a] = Stream();
            p.train(b, 8); p.train(b, 8);
        }
        for (int k = 0; k < 3; ++k) {      // read-outs, then an update in place or one after another, not on the same stream
            Program p(net);
            p.gets_ordered = false;
            hipStream_t a = new_stream(), b = new_stream();
            p.init(a); p.predict(a, 3); p.train(a, 8);
            if (k == 0) { p.get(a); p.train(b, 8); }
            if (k == 1) { p.get(a); p.get(b); p.train(b, 8); }
            if (k == 2) { p.predict(a, 3); p.get(b); p.train(a, 8); p.predict(a, 3); p.train(a, 8); }
        }
        for (int seed = 0; seed < 20; ++seed) {
            Program p(net);
            rng_state = 977u * (unsigned)seed + 5u;
            std::vector<hipStream_t> s = {nullptr, new_stream(), new_stream(), new_stream()};
            const int width = 1 + any(4);
            p.init(s[any(width)]);
            for (int k = 0; k < 60; ++k) {
                hipStream_t t = s[any(width)];
                const int what = any(14);
                if (what < 6) p.predict(t, 1 + any(64));
                else if (what < 10) p.train(t, 1 + any(16));
                else if (what == 10) p.get(t);
                else if (what == 11) p.init(t, any(2) != 0);
                else if (width > 1) {                   // a stream ends, another one takes its place
                    const int i = 1 + any(width - 1);
                    p.over(s[i]);
                    (void)hipStreamDestroy(s[i]);
                    s[i] = new_stream();
                }
            }
        }
    }
}

// A stream under capture gets no launch that carries an event, and the fences all the same.
static void capture_check() {
    Program p("small");
    hipStream_t a = new_stream(), b = new_stream();
    p.init(a);
    for (int k = 0; k < 3; ++k) {
        streams[b].capturing = true;
        p.predict(b, 5); p.get(b); p.train(b, 8); p.predict(b, 64);
        streams[b].capturing = false;
        p.train(a, 8); p.train(a, 8);
    }
}

// Predictions leave no event behind, whatever stream they are on: one per publication, before the first of them; an update's event
// rides on its last launch, and it does not wait for predictions of the parameters that it reads itself.
static void packets_check() {
    for (const char *net : {"small", "large", "paper3"}) {
        Program p(net);
        hipStream_t a = new_stream(), b = new_stream();
        p.init(a);
        for (int k = 0; k < 10; ++k) {
            const int before = records;
            for (int j = 0; j < 5; ++j) p.predict(b, 1 + 6 * k);
            if (records != before + (k > 0)) PROBLEM("%d events recorded for five predictions", records - before);
            const int latest = (int)ops.size() - 1, marked = records;
            p.train(a, 8);
            if (records != marked) PROBLEM("an update recorded events behind its launches");
            if (latest < (int)ops.back().before.size() && ops.back().before[latest]) PROBLEM("an update waits for predictions of the parameters that it reads");
        }
    }
}

// A scheduler's tick only enqueues, from the first one on, whichever way its network takes the frames: nothing is allocated, no
// stream is waited for, no other stream used than the scheduler's two.
static void ticks_check() {
    for (const char *net : {"small", "large", "paper3"})
        for (bool generic : {false, true}) {
            Program p(net);
            p.init(nullptr);
            const std::map<hipStream_t, Stream> before = streams;
            ga3c_sched_config cfg;
            memset(&cfg, 0, sizeof(cfg));
            cfg.t_max = 5; cfg.predict_cap = 16; cfg.train_min = 10; cfg.train_cap = 40; cfg.hp = p.hp;
            ga3c_sched *s = nullptr;
            if (ga3c_sched_create(p.ctx, &cfg, &s) != GA3C_OK) { PROBLEM("sched_create: %s", ga3c_sched_last_error()); return; }
            given.clear();
            for (const auto &x : streams) if (!before.count(x.first)) given.insert(x.first);
            if (generic) ga3c_use_generic_kernels(p.ctx, 1);
            const int32_t actions[5] = {0, 1, 2, 3, 4};
            const float rewards[5] = {0, 0, 1, 0, 0};
            const uint8_t dones[5] = {0, 0, 0, 0, 1};
            for (int k = 0; k < 12; ++k) {
                for (int a = 0; a < 20; ++a) {
                    if (ga3c_sched_submit_predict(s, a, address(a), 0.5f) != GA3C_OK) PROBLEM("submit_predict");
                    if (ga3c_sched_submit_segment(s, a, address(a), 1 + (a + k) % 5, actions, rewards, dones, 0.f, 0) != GA3C_OK) PROBLEM("submit_segment");
                }
                in_call = true;
                int predicted = 0, trained = 0;
                if (ga3c_sched_tick(s, &predicted, &trained) != GA3C_OK) PROBLEM("tick: %s", ga3c_sched_last_error());
                in_call = false;
                if (predicted < 1 || trained < 1) PROBLEM("a tick of %d predictions and %d trained frames", predicted, trained);
            }
            ga3c_sched_destroy(s);
        }
}

// Host memory that runs out while requests and segments are handed in is an error code, with nothing or everything queued.
static void memory_check() {
    Program p("small");
    p.init(nullptr);
    ga3c_sched_config cfg;
    memset(&cfg, 0, sizeof(cfg));
    cfg.t_max = 5; cfg.predict_cap = 16; cfg.train_min = 160; cfg.train_cap = 160; cfg.hp = p.hp;
    ga3c_sched *s = nullptr;
    if (ga3c_sched_create(p.ctx, &cfg, &s) != GA3C_OK) { PROBLEM("sched_create: %s", ga3c_sched_last_error()); return; }
    const int32_t actions[5] = {0, 1, 2, 3, 4}, agents[3] = {0, 1, 2};
    const float rewards[5] = {0, 0, 1, 0, 0}, uniforms[3] = {0.1f, 0.2f, 0.3f};
    const uint8_t dones[5] = {0, 0, 0, 0, 1}, *frames[3] = {address(0), address(1), address(2)};
    long requests = 0, segments = 0, refused = 0;
    for (int k = 0; k < 600; ++k)
        for (int left = 0; left < 6; ++left) {          // the first, second, ... allocation of the call fails
            const int what = k % 3;
            memory_left = left;
            int rc;
            try {
                rc = what == 0   ? ga3c_sched_submit_predict(s, k, address(0), 0.5f)
                     : what == 1 ? ga3c_sched_submit_predict_many(s, 3, agents, frames, uniforms)
                                 : ga3c_sched_submit_segment(s, k, address(0), 1 + k % 5, actions, rewards, dones, 0.f, 0);
            } catch (...) { memory_left = -1; PROBLEM("an exception came out of a call"); return; }
            memory_left = -1;
            if (rc == GA3C_OK) { requests += what == 0 ? 1 : what == 1 ? 3 : 0; segments += what == 2; }
            else if (rc != GA3C_ENOMEM) PROBLEM("code %d for memory that ran out", rc);
            else ++refused;
            ga3c_sched_stats st;
            ga3c_sched_get_stats(s, &st);
            if (st.predict_queue != requests || st.train_queue != segments) PROBLEM("%ld requests and %ld segments queued, %ld and %ld accepted",
                                                                                    (long)st.predict_queue, (long)st.train_queue, requests, segments);
        }
    if (refused < 10) PROBLEM("memory ran out %ld times only", refused);
    for (int total = 0, none = 0; none < 3;) {           // what was accepted goes through
        int predicted = 0, trained = 0;
        if (ga3c_sched_tick(s, &predicted, &trained) != GA3C_OK) { PROBLEM("tick: %s", ga3c_sched_last_error()); break; }
        total += predicted;
        none = predicted || trained ? 0 : none + 1;
        if (none == 3 && total != requests) PROBLEM("%d of %ld requests went through", total, requests);
    }
    ga3c_sched_destroy(s);
}

// A tick that fails half way has launched kernels that read the slot's lists and write into its results: the next tick, which
// takes the same slot, must find them over.
static void failures_check() {
    for (const char *net : {"small", "large", "paper3"})
        for (const bool training : {false, true})
            for (int what = 0; what < 12; ++what) {        // the event, or the first, second, .. launch
                Program p(net);
                p.init(nullptr);
                ga3c_sched_config cfg;
                memset(&cfg, 0, sizeof(cfg));
                cfg.t_max = 5; cfg.predict_cap = 16; cfg.train_min = 10; cfg.train_cap = 40; cfg.hp = p.hp;
                ga3c_sched *s = nullptr;
                if (ga3c_sched_create(p.ctx, &cfg, &s) != GA3C_OK) { PROBLEM("sched_create: %s", ga3c_sched_last_error()); return; }
                const int32_t actions[5] = {0, 1, 2, 3, 4};
                const float rewards[5] = {0, 0, 1, 0, 0};
                const uint8_t dones[5] = {0, 0, 0, 0, 1};
                auto submit = [&] {
                    for (int a = 0; a < 4; ++a)
                        if ((training ? ga3c_sched_submit_segment(s, a, address(a), 5, actions, rewards, dones, 0.f, 0)
                                      : ga3c_sched_submit_predict(s, a, address(a), 0.5f)) != GA3C_OK) PROBLEM("submit");
                };
                auto ticked = [&] { int predicted = 0, trained = 0; return ga3c_sched_tick(s, &predicted, &trained) == GA3C_OK ? predicted + trained : -1; };
                // predictions of new parameters and the first update record events of the context's own
                submit();
                if (ticked() < 0 || ga3c_sched_drain(s) != GA3C_OK) PROBLEM("a first tick: %s", ga3c_sched_last_error());
                ga3c_prediction out[16];
                if (ga3c_sched_poll(s, out, 16) != (training ? 0 : 4)) PROBLEM("results of the first tick");
                submit();
                const size_t first = ops.size();
                (what ? launches_left : records_left) = what ? what - 1 : 0;
                const int got = ticked();
                const bool failed = (what ? launches_left : records_left) < 0;
                launches_left = records_left = -1;
                if ((got < 0) != failed) PROBLEM("%s network, %s: a call failed and the tick says %d", net, training ? "update" : "prediction", got);
                if (got < 0) {
                    for (size_t i = first; i < ops.size(); ++i)
                        if (!(i < host.size() && host[i])) { PROBLEM("%s network, a failed %s: %s may still run", net, training ? "update" : "prediction", ops[i].name.c_str()); break; }
                    if (ticked() < 0) PROBLEM("the tick behind a failed one: %s", ga3c_sched_last_error());
                    if (ga3c_sched_drain(s) != GA3C_OK || ga3c_sched_poll(s, out, 16) != (training ? 0 : 4)) PROBLEM("%s network: a failed call lost requests", net);
                }
                ga3c_sched_destroy(s);
            }
}

// The workspace of partial sums, which a context allocates last: enough for an update of every size up to the capacity, on both
// kinds of kernels, and for a few frames of the any-size layers no more than the bands that they are cut into.
static void workspace_check() {
    for (const char *net : {"small", "large", "paper1", "paper2", "paper3", "paper4"})
        for (int math : {0, 1})
            for (int cap : {1, 5, 40, 140, 600, 1280}) {
                ga3c_net_desc d = net_desc(net);
                d.math = math;
                ga3c_ctx *ctx = nullptr;
                if (ga3c_create(&d, 0, cap, &ctx) != GA3C_OK) { PROBLEM("create: %s", ga3c_last_error()); continue; }
                // 128 bands, a few more where they don't come out even, of three layers; any other sum takes no more than the parameters
                const size_t most = 4 * (160 * (32 * 257 + 32 * 513 + 64 * 513) + 2 * ga3c_params_count(ctx));
                if (!strncmp(net, "paper", 5) && cap <= 5 && last_bytes > most) PROBLEM("%s, %d frames: %zu bytes of workspace", net, cap, last_bytes);
                const ga3c_hparams hp = {0.99f, 0.01f, 1.f, 0.f, 1e-4f, 0.99f, 0.1f, 40.f};
                for (int generic : {0, 1}) {
                    ga3c_use_generic_kernels(ctx, generic);
                    for (int B = 1; B <= cap; ++B) {
                        if (ga3c_train_step(ctx, address(0), (const int32_t *)address(1), (const float *)address(2), address(3), nullptr, B, 1, &hp, nullptr, nullptr) != GA3C_OK) {
                            PROBLEM("%s, math %d, capacity %d: an update of %d frames: %s", net, math, cap, B, ga3c_last_error());
                            break;
                        }
                        if (B % 20 == 0 || B == cap) {             // the order of these launches is not what is looked at
                            ops.clear(); host.clear(); streams[nullptr] = Stream();
                            for (auto &e : events) e.second.seen.clear();
                        }
                    }
                }
                ga3c_destroy(ctx);
            }
}

// What a context keeps of the any-size layers' filters: with operands rounded to bfloat16 one term of two bytes per weight and
// purpose, which is less than the terms, or the floats in another order, of the exact variant.
static void fragments_check() {
    for (int train : {0, 5}) {
        size_t bytes[2];
        for (int math : {0, 1}) {
            ga3c_net_desc d = net_desc("paper3");
            d.math = math;
            d.fc_units = 16;                              // too few for the fc layer's operands to be kept
            const size_t before = device_bytes;
            ga3c_ctx *ctx = nullptr;
            if (ga3c_create(&d, 1, train, &ctx) != GA3C_OK) { PROBLEM("create: %s", ga3c_last_error()); return; }
            bytes[math] = device_bytes - before;
            ga3c_destroy(ctx);
            if (device_bytes != before) PROBLEM("%zu bytes of device memory left behind", device_bytes - before);
        }
        const size_t weights = 32 * 256 + 32 * 512 + 64 * 512;
        // two copies: the byte layer's terms (6 bytes a weight) and the others' floats against one term of each
        if (train == 0 && bytes[0] - bytes[1] < 2 * (6 * 8192 + 4 * (weights - 8192) - 2 * weights)) PROBLEM("%zu bytes exact, %zu rounded", bytes[0], bytes[1]);
        if (bytes[1] >= bytes[0]) PROBLEM("%d frames: %zu bytes exact, %zu rounded", train, bytes[0], bytes[1]);
    }
}

// Two batches in flight, of which the second is over by the time that it is looked at and the first was not yet: results come
// oldest first all the same.
static void order_check() {
    Program p("small");
    p.init(nullptr);
    ga3c_sched_config cfg;
    memset(&cfg, 0, sizeof(cfg));
    cfg.t_max = 5; cfg.predict_cap = 4; cfg.train_min = 10; cfg.train_cap = 40; cfg.hp = p.hp;
    ga3c_sched *s = nullptr;
    if (ga3c_sched_create(p.ctx, &cfg, &s) != GA3C_OK) { PROBLEM("sched_create: %s", ga3c_sched_last_error()); return; }
    for (int round = 0; round < 6; ++round) {              // every slot comes first once
        int predicted = 0;
        for (int a = 0; a < 8; ++a)
            if (ga3c_sched_submit_predict(s, a, address(a), 0.5f) != GA3C_OK) PROBLEM("submit_predict");
        for (int k = 0; k < 2; ++k) {
            queries_left = 0;                              // the tick's own look at the first batch
            if (ga3c_sched_tick(s, &predicted, nullptr) != GA3C_OK || predicted != 4) PROBLEM("tick: %d", predicted);
        }
        ga3c_prediction out[16];
        queries_left = 0;
        int got = ga3c_sched_poll(s, out, 16);
        queries_left = -1;
        while (got < 8) {
            const int more = ga3c_sched_poll(s, out + got, 16 - got);
            if (more <= 0) { PROBLEM("%d of 8 results", got); break; }
            got += more;
        }
        for (int a = 0; a < got; ++a)
            if (out[a].agent != a) { PROBLEM("result %d is agent %d's", a, out[a].agent); break; }
    }
    ga3c_sched_destroy(s);
}

int main(int argc, char **argv) {
    streams[nullptr] = Stream();
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "streams") streams_check();
    else if (what == "capture") capture_check();
    else if (what == "packets") packets_check();
    else if (what == "ticks") ticks_check();
    else if (what == "memory") memory_check();
    else if (what == "failures") failures_check();
    else if (what == "order") order_check();
    else if (what == "workspace") workspace_check();
    else if (what == "fragments") fragments_check();
    else PROBLEM("no such check");
    printf("%zu launches, %d problems\n", ops.size(), problems);
    return problems ? 1 : 0;
}
