// The order of a decoder state's device work, checked without a device: a model
// of the HIP runtime's streams, events and captures stands in for the library,
// and the scenarios below drive the C ABI on it.  Every stream and event carries
// a vector clock; each launch, copy or fill of a state must come after the one
// before it, whatever streams they are on.
//   order_driver <scenario>   prints each failed expectation and "failures N".
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "dc.h"

static int g_failures = 0;
static void expect(bool ok, const char* what)
{
    if (ok) return;
    std::printf("FAILED: %s\n", what);
    g_failures++;
}

// ------------------------------------------------------- the runtime's model

struct Clock {
    std::map<int, long> t;
    void merge(const Clock& o)
    {
        for (auto& [k, v] : o.t)
            if (t[k] < v) t[k] = v;
    }
    bool covers(const Clock& o) const
    {
        for (auto& [k, v] : o.t) {
            auto it = t.find(k);
            if (it == t.end() || it->second < v) return false;
        }
        return true;
    }
};
static std::set<int> g_ended;   // queues of ended threads
struct Queue {   // what a stream handle names
    int id;
    Clock c;
    bool cap = false, bad = false;   // being captured; that capture is invalid
    bool of_thread = false;
    Queue() : id(next()++) {}
    ~Queue()
    {
        if (of_thread) g_ended.insert(id);
    }
    static int& next()
    {
        static int n = 0;
        return n;
    }
};
struct ihipStream_t {
    Queue* q;
};
struct ihipEvent_t {
    Clock c;
    int queue = -1;
    bool cap = false;
};
struct ihipGraph {
    int ops;
};
struct hipGraphExec {
    int ops;
};

static Queue g_default;
static Clock g_host, g_last;                 // what the host has waited for; the last device operation
static std::vector<ihipStream_t*> g_free;    // destroyed handles, the next ones to be handed out again
static std::vector<Queue*> g_captured;
static int g_unordered = 0, g_ops = 0, g_cap_ops = 0, g_fail_waits = 0, g_fail_syncs = 0, g_fail_queries = 0;
static thread_local hipError_t t_err = hipSuccess;
static std::map<char*, size_t> g_mem;

static hipError_t ret(hipError_t e)
{
    if (e != hipSuccess) t_err = e;
    return e;
}
static Queue& queue(hipStream_t s)
{
    static thread_local Queue per_thread;
    per_thread.of_thread = true;
    if (!s) return g_default;
    if (s == hipStreamPerThread) return per_thread;
    return *s->q;
}
static hipError_t op(hipStream_t s)
{
    Queue& q = queue(s);
    if (q.cap) {
        g_cap_ops++;
        return hipSuccess;
    }
    q.c.merge(g_host);
    if (!q.c.covers(g_last)) g_unordered++;
    q.c.merge(g_last);
    q.c.t[q.id]++;
    g_last = q.c;
    g_ops++;
    return hipSuccess;
}

extern "C" {
hipError_t hipMalloc(void** p, size_t n)
{
    *p = std::calloc(1, n);
    g_mem[(char*)*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    g_mem.erase((char*)p);
    std::free(p);
    return hipSuccess;
}
static std::map<char*, size_t>::iterator allocation(const void* p)
{
    auto it = g_mem.upper_bound((char*)p);
    if (it == g_mem.begin()) return g_mem.end();
    --it;
    return (char*)p < it->first + it->second ? it : g_mem.end();
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p)
{
    if (allocation(p) == g_mem.end()) return ret(hipErrorInvalidValue);
    std::memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p)
{
    auto it = allocation(p);
    if (it == g_mem.end()) return ret(hipErrorNotFound);
    *base = it->first;
    *size = it->second;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceSynchronize() { return g_host.merge(g_last), hipSuccess; }
hipError_t hipGetLastError()
{
    const hipError_t e = t_err;
    t_err = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "an error of the model"; }
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    static char mem[64];
    return *p = mem, hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemcpyToSymbol(const void*, const void*, size_t, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyFromSymbol(void*, const void*, size_t, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t s) { return op(s); }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t s) { return op(s); }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t s) { return op(s); }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    if (g_free.empty()) {
        *s = new ihipStream_t;
    } else {
        *s = g_free.back();
        g_free.pop_back();
    }
    (*s)->q = new Queue;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return g_free.push_back(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return g_host.merge(queue(s).c), hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* out)
{
    if (g_fail_queries > 0) return g_fail_queries--, ret(hipErrorStreamCaptureImplicit);
    *out = queue(s).cap ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    queue(s).cap = true;
    queue(s).bad = false;
    g_captured = {&queue(s)};
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g)
{
    *g = new ihipGraph{g_cap_ops};
    for (Queue* q : g_captured) q->cap = false;
    g_captured.clear();
    return queue(s).bad ? ret(hipErrorStreamCaptureInvalidated) : hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t)
{
    *x = new hipGraphExec{g->ops};
    return hipSuccess;
}
hipError_t hipGraphGetNodes(hipGraph_t g, hipGraphNode_t*, size_t* n) { return *n = g->ops, hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return op(s); }
hipError_t hipGraphDestroy(hipGraph_t g) { return delete g, hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return delete x, hipSuccess; }

hipError_t hipEventCreate(hipEvent_t* e) { return *e = new ihipEvent_t, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete e, hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0.f, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    e->cap = queue(s).cap;
    e->queue = queue(s).id;
    e->c = queue(s).c;
    e->c.merge(g_host);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    for (Queue* q : g_captured) q->bad = true;   // not allowed while the thread captures
    if (!g_captured.empty()) return ret(hipErrorStreamCaptureUnsupported);
    if (g_fail_syncs > 0) return g_fail_syncs--, ret(hipErrorUnknown);
    g_host.merge(e->c);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    Queue& q = queue(s);
    if (g_fail_waits > 0) return g_fail_waits--, ret(hipErrorUnknown);
    if (q.cap && !e->cap) return q.bad = true, ret(hipErrorStreamCaptureIsolation);
    if (!q.cap && e->cap) {   // joins the capture
        q.cap = true;
        g_captured.push_back(&q);
    }
    if (g_ended.count(e->queue)) return hipSuccess;   // taken for done, though the thread may still be ending
    q.c.merge(e->c);
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { return (void**)&g_ops; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
static thread_local struct {
    dim3 g, b;
    size_t n;
    hipStream_t s;
} t_config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t n, hipStream_t s) { return t_config = {g, b, n, s}, hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* s)
{
    *g = t_config.g, *b = t_config.b, *n = t_config.n, *s = t_config.s;
    return hipSuccess;
}
}

// ---------------------------------------------------------------- scenarios

static const int kChunk = 8;

struct Fixture {
    dc_state* s = nullptr;
    hipStream_t own = nullptr, a = nullptr, b = nullptr;
    int32_t* tok = nullptr;
    float *pcm = nullptr, *f0 = nullptr;
    explicit Fixture(bool source = false)
    {
        dc_cfg c{};
        c.abi_version = DC_ABI_VERSION;
        c.vocab = 256, c.embed = 64, c.frames_per_token = 1, c.n_pre = 1, c.pre_kernel = 3, c.n_stages = 2;
        c.up_rate[0] = 2, c.up_rate[1] = 2;
        c.channels[0] = 64, c.channels[1] = 32, c.channels[2] = 16;
        c.n_rb = 1, c.rb_kernel[0] = 3, c.n_dil = 1, c.dil[0] = 1;
        c.head_kernel = 7, c.n_fft = 16, c.hop = 4, c.lrelu_slope = 0.1f;
        c.dtype = DC_F32, c.batch = 1, c.chunk_tokens = kChunk, c.max_tokens = kChunk;
        c.sine_amp = 0.1f, c.noise_std = 0.003f, c.voiced_threshold = 10.0f, c.sample_rate = 24000.0f;
        c.n_harmonics = source ? 8 : 0;
        (void)hipStreamCreateWithFlags(&own, 0);
        (void)hipStreamCreateWithFlags(&a, 0);
        (void)hipStreamCreateWithFlags(&b, 0);
        c.hip_stream = own;
        std::vector<float> blob((size_t)dc_blob_floats(&c), 0.0f);
        expect(dc_init(blob.data(), blob.size() * 4, &c, &s) == DC_OK, "dc_init");
        (void)hipMalloc((void**)&tok, kChunk * 4);
        (void)hipMalloc((void**)&f0, kChunk * 4);
        (void)hipMalloc((void**)&pcm, kChunk * dc_samples_per_token(&c) * 4);
        g_unordered = 0;
    }
    ~Fixture() { dc_free(s); }
    dc_status on(hipStream_t st, int n = kChunk) { return dc_decode_chunk_on(s, st, tok, nullptr, n, pcm); }
    dc_status home(int n = kChunk) { return dc_decode_chunk(s, tok, n, pcm); }
};

// Calls of every kind on every stream, none waited for.
static void several_streams()
{
    Fixture f;
    const hipStream_t order[] = {f.a, f.b, f.own, nullptr, f.a, f.a, nullptr, f.b, f.own, f.own, f.b};
    int i = 0;
    for (hipStream_t st : order) {
        expect(f.on(st, i % 3 ? kChunk : 3) == DC_OK, "a call on a stream");
        if (i % 4 == 1) expect(f.home() == DC_OK, "a call on the state's stream");
        if (i % 4 == 2) expect(dc_reset_stream(f.s, 0) == DC_OK, "a stream's reset");
        if (i == 6) expect(dc_sync(f.s) == DC_OK, "a wait");
        if (i == 7) expect(dc_reset(f.s) == DC_OK, "a reset");
        i++;
    }
    expect(g_unordered == 0, "every call comes after the one before it");
}

// Work that the caller puts on the state's own stream, with dc_settle around the calls.
static void settle()
{
    Fixture f;
    for (hipStream_t st : {f.a, f.b, f.b}) {
        expect(dc_settle(f.s) == DC_OK && f.on(st) == DC_OK && dc_settle(f.s) == DC_OK, "a settled call");
        (void)op(f.own);   // the caller's
        if (st == f.a) expect(dc_sync(f.s) == DC_OK, "a wait");
        (void)op(f.own);
    }
    expect(dc_settle(f.s) == DC_OK && f.on(f.a) == DC_OK, "a last call");
    expect(g_unordered == 0, "the caller's work on the state's stream and the calls are in order");
}

// A stream that is being captured cannot wait for a call outside the capture.
static void capture()
{
    {
        Fixture f;
        hipGraph_t g;
        expect(f.on(f.a) == DC_OK, "a call");
        (void)hipStreamBeginCapture(f.own, hipStreamCaptureModeThreadLocal);
        const int before = g_cap_ops;
        expect(f.home() == DC_ESTATE, "refused: the state's stream, being captured, has an outside call to wait for");
        expect(dc_settle(f.s) == DC_ESTATE, "so is settling");
        expect(f.on(f.b) == DC_OK, "another stream's call is not in the way of the capture");
        expect(f.on(f.own) == DC_ESTATE, "refused on the state's stream by name");
        expect(g_cap_ops == before, "nothing was captured");
        expect(hipStreamEndCapture(f.own, &g) == hipSuccess, "the capture stayed valid");
        expect(dc_settle(f.s) == DC_OK && f.home() == DC_OK, "and the state works on");
        // a captured stream of the caller's, and a captured state's stream that has had work
        (void)hipStreamBeginCapture(f.a, hipStreamCaptureModeThreadLocal);
        expect(f.on(f.a) == DC_ESTATE && g_cap_ops == before, "refused on a stream being captured");
        expect(hipStreamEndCapture(f.a, &g) == hipSuccess, "that capture stayed valid");
        (void)hipStreamBeginCapture(f.own, hipStreamCaptureModeThreadLocal);
        expect(f.home() == DC_OK && g_cap_ops > before, "a settled state's stream can be captured");
        expect(f.on(f.a) == DC_ESTATE, "refused: other streams would join the capture");
        expect(hipStreamEndCapture(f.own, &g) == hipSuccess, "that capture stayed valid too");
        expect(f.on(f.a) == DC_OK && f.home() == DC_OK, "after it both work");
        expect(g_unordered == 0, "in order");
    }
    Fixture f(true);   // the entry point for captures
    hipGraph_t g;
    auto call = [&] { return dc_decode_chunk_f0_static(f.s, f.tok, f.f0, kChunk, f.pcm); };
    expect(dc_decode_chunk_on(f.s, f.a, f.tok, f.f0, kChunk, f.pcm) == DC_OK, "a call");
    (void)hipStreamBeginCapture(f.own, hipStreamCaptureModeThreadLocal);
    expect(call() == DC_ESTATE, "refused before dc_settle");
    expect(hipStreamEndCapture(f.own, &g) == hipSuccess, "the capture stayed valid");
    expect(dc_settle(f.s) == DC_OK, "settled");
    (void)hipStreamBeginCapture(f.own, hipStreamCaptureModeThreadLocal);
    const int before = g_cap_ops;
    expect(call() == DC_OK && g_cap_ops > before, "captured after it");
    expect(hipStreamEndCapture(f.own, &g) == hipSuccess, "a valid capture");
}

// A wait that cannot be enqueued is reported and stays due.
static void failing_wait()
{
    Fixture f;
    for (int kind = 0; kind < 3; kind++) {
        expect(f.on(f.a) == DC_OK, "a call");
        g_fail_waits = g_fail_syncs = 1;
        const dc_status st = kind == 0 ? f.home() : kind == 1 ? dc_settle(f.s) : dc_reset_stream(f.s, 0);
        g_fail_waits = g_fail_syncs = 0;
        expect(st == DC_EDEVICE, "reported");
        expect(dc_reset(f.s) == DC_OK && f.home() == DC_OK, "a reset clears it");
        expect(g_unordered == 0, "after the call that was to be waited for");
    }
}

// One handle value, several streams: the per-thread stream of two threads, and a
// destroyed stream's handle handed out again.
static void same_handle()
{
    Fixture f;
    for (int i = 0; i < 4; i++) {
        if (i % 2) std::thread([&] { expect(f.on(hipStreamPerThread) == DC_OK, "a call on a thread's stream"); }).join();
        else expect(f.on(hipStreamPerThread) == DC_OK, "a call on this thread's stream");
    }
    std::thread([&] { expect(f.on(hipStreamPerThread) == DC_OK, "a call on another thread's stream"); }).join();
    expect(f.home() == DC_OK, "a call on the state's stream");
    std::thread([&] { expect(f.on(hipStreamPerThread) == DC_OK, "a call on another thread's stream"); }).join();
    expect(f.on(f.a) == DC_OK, "a call on a stream");
    expect(g_unordered == 0, "the per-thread streams are in order");
    hipStream_t old = nullptr;
    for (int i = 0; i < 3; i++) {
        hipStream_t st;
        (void)hipStreamCreateWithFlags(&st, 0);
        expect(!old || st == old, "(the handle is used again)");
        expect(f.on(st) == DC_OK, "a call on a new stream");
        (void)hipStreamDestroy(old = st);
    }
    expect(g_unordered == 0, "the streams of one handle are in order");
}

// An error of the caller's own is neither the call's nor taken from the caller.
static void callers_error()
{
    Fixture f;
    for (int i = 0; i < 4; i++) {
        t_err = hipErrorOutOfMemory;
        expect((i % 2 ? f.home() : f.on(f.a)) == DC_OK, "a replay after a failed call of the caller's");
        expect(hipGetLastError() == hipErrorOutOfMemory, "whose error is still there");
    }
    // nor does a query that the runtime refuses leave one (the default stream's, while another is captured)
    g_fail_queries = 1;
    expect(f.on(nullptr, 3) == DC_OK && hipGetLastError() == hipSuccess, "direct launches after a refused query");
    expect(dc_sync(f.s) == DC_OK, "a sound state");
}

int main(int argc, char** argv)
{
    const std::string which = argc > 1 ? argv[1] : "";
    const std::map<std::string, void (*)()> all = {
        {"several_streams", several_streams}, {"settle", settle}, {"capture", capture}, {"failing_wait", failing_wait},
        {"same_handle", same_handle}, {"callers_error", callers_error}};
    if (all.count(which)) all.at(which)();
    else expect(false, "unknown scenario");
    std::printf("failures %d\n", g_failures);
    return g_failures ? 1 : 0;
}
