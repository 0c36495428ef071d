// The host runtime (dock_runtime.cpp) on a CPU, for tests of its streams, captures and
// launch shapes: the HIP calls it makes and the kernel launchers are replaced by a model
// of streams.  Device memory is host memory; a launch computes nothing, it is one entry
// of its stream's queue and of the log.
//
// Queues run in order; an event wait holds its queue until the record it saw has run.
// A held stream (stub_hold) runs nothing, as a stream whose earlier work is not done.
// stub_fail(name, n) makes the n-th call from now on of that HIP function fail.
#include <algorithm>
#include <cstdlib>
#define __align__(n)
#define HIP_SYMBOL(x) (x)
#include "dock_runtime.cpp"

#include <deque>
#include <set>
#include <sstream>

namespace {

using Token = std::shared_ptr<int>;  // a record: 0 enqueued, 1 run, 2 inside a capture

struct Op {
    Token wait, record;
};
struct Event {
    Token last;
    hipStream_t on = nullptr;
    size_t at = 0;  // place in the log
};
struct Capture {
    std::set<hipStream_t> members;   // the origin and the streams forked from it
    std::set<hipStream_t> unjoined;  // those with work that no other member waits for
};

std::map<hipStream_t, std::deque<Op>> g_queue;
std::set<hipStream_t> g_held;
std::map<hipStream_t, Capture> g_capture;  // by origin stream
std::set<hipStream_t> g_caller_capture;    // streams a caller captures (stub_capture)
std::map<hipGraphExec_t, Token> g_exec;    // last launch of each
std::map<std::string, int> g_fail;
int g_stay[kNumBins];  // orientations that stay in the probes of a pocket's bounds
std::string g_log;
std::string g_log_out;
uintptr_t g_next = 0x1000;
size_t g_allocs = 0;

bool fails(const char *name) {
    auto it = g_fail.find(name);
    if (it == g_fail.end()) return false;
    if (--it->second > 0) return false;
    g_fail.erase(it);
    return true;
}
#define STUB_FAIL(name) \
    if (fails(name)) return hipErrorUnknown

Capture *capture_of(hipStream_t s) {
    for (auto &kv : g_capture)
        if (kv.second.members.count(s)) return &kv.second;
    return nullptr;
}

void run_queues() {
    for (bool moved = true; moved;) {
        moved = false;
        for (auto &kv : g_queue) {
            if (g_held.count(kv.first)) continue;
            while (!kv.second.empty()) {
                Op &o = kv.second.front();
                if (o.wait && *o.wait == 0) break;
                if (o.record && *o.record == 0) *o.record = 1;
                kv.second.pop_front();
                moved = true;
            }
        }
    }
}

void note(const std::string &what, hipStream_t s) {
    std::ostringstream o;
    o << what << " stream=" << (uintptr_t)s << (capture_of(s) ? " captured" : "") << "\n";
    g_log += o.str();
}

hipError_t launched(const std::string &what, hipStream_t s) {
    STUB_FAIL("launch");
    note(what, s);
    if (Capture *c = capture_of(s)) c->unjoined.insert(s);
    else g_queue[s].push_back({});
    return hipSuccess;
}

template <class... T>
std::string text(T... v) {
    std::ostringstream o;
    (o << ... << v);
    return o.str();
}

}  // namespace

// ---------------------------------------------------------------------------
// HIP
extern "C" {
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "stub error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    std::memset((void *)p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950:stub");
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **out, const void *sym) { *out = (void *)sym; return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)288 << 30; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
    STUB_FAIL("hipMalloc");
    *p = std::calloc(1, n ? n : 1);
    g_allocs += 1;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
    if (p) {
        std::free(p);
        g_allocs -= 1;
        note("free", nullptr);
    }
    return hipSuccess;
}
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return hipMalloc(p, n); }
hipError_t hipFreeAsync(void *p, hipStream_t s) { note("freeAsync", s); std::free(p); g_allocs -= p != nullptr; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n ? n : 1); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
    std::memcpy(d, s, n);
    return launched("memcpy", st);
}
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipDeviceSynchronize() { run_queues(); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    note("synchronize", s);
    run_queues();
    return g_queue[s].empty() ? hipSuccess : hipErrorLaunchTimeOut;  // would hang
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    STUB_FAIL("hipStreamCreateWithFlags");
    *s = (hipStream_t)(g_next++);
    return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) {
    run_queues();
    return g_queue[s].empty() ? hipSuccess : hipErrorNotReady;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = (hipEvent_t) new Event();
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    STUB_FAIL("hipEventRecord");
    Event *ev = (Event *)e;
    if (capture_of(s)) {
        ev->last = std::make_shared<int>(2);
    } else {
        ev->last = std::make_shared<int>(0);
        g_queue[s].push_back({nullptr, ev->last});
    }
    ev->on = s;
    ev->at = g_log.size();
    note("record", s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    STUB_FAIL("hipStreamWaitEvent");
    Event *ev = (Event *)e;
    note("wait", s);
    if (!ev->last) return hipSuccess;  // never recorded
    if (*ev->last == 2) {
        Capture *c = capture_of(ev->on);
        if (!c) return hipErrorCapturedEvent;  // of a capture that has ended
        c->unjoined.erase(ev->on);
        c->members.insert(s);
        c->unjoined.insert(s);
        return hipSuccess;
    }
    if (capture_of(s)) return hipErrorStreamCaptureIsolation;
    g_queue[s].push_back({ev->last, nullptr});
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    Event *ev = (Event *)e;
    run_queues();
    if (!ev->last || *ev->last == 1) return hipSuccess;
    return *ev->last == 2 ? hipErrorCapturedEvent : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return hipEventQuery(e); }
// A launch takes 1 ms, a selection of 16 waves 0.5 by itself and 2 beside a sweep.
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) {
    const std::string part = g_log.substr(((Event *)a)->at, ((Event *)b)->at - ((Event *)a)->at);
    const bool beside = part.find("dock bin") != std::string::npos;
    std::istringstream in(part);
    *ms = 0.f;
    for (std::string line; std::getline(in, line);) {
        if (line.find("blocks=") == std::string::npos) continue;
        const bool s16 = line.find("select") == 0 && line.find("waves=16") != std::string::npos;
        *ms += !s16 ? 1.f : beside ? 2.f : 0.5f;
    }
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) {
    *st = g_caller_capture.count(s) || capture_of(s) ? hipStreamCaptureStatusActive
                                                     : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    note("beginCapture", s);
    if (g_caller_capture.count(s) || capture_of(s)) return hipErrorIllegalState;
    g_capture[s].members.insert(s);
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
    g_capture[s].unjoined.erase(s);
    const bool open = !g_capture[s].unjoined.empty();
    g_capture.erase(s);
    *g = open ? nullptr : (hipGraph_t)0x1;
    return open ? hipErrorStreamCaptureUnjoined : hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *x = (hipGraphExec_t)(g_next++);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
    run_queues();
    Token t = g_exec[x];
    note(t && *t == 0 ? "graph destroyed in flight" : "graph destroyed", nullptr);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
    if (g_caller_capture.count(s)) return hipErrorIllegalState;
    g_exec[x] = std::make_shared<int>(0);
    g_queue[s].push_back({nullptr, g_exec[x]});
    return launched("graph", s);
}

// ---------------------------------------------------------------------------
// Of the tests
const char *stub_log() {
    g_log_out = g_log;
    g_log.clear();
    return g_log_out.c_str();
}
void stub_hold(void *s, int on) {
    if (on) {
        g_queue[(hipStream_t)s].push_back({});
        g_held.insert((hipStream_t)s);
    } else {
        g_held.erase((hipStream_t)s);
    }
}
int stub_idle(void *s) {  // whether everything enqueued on the stream has run
    run_queues();
    return g_queue[(hipStream_t)s].empty();
}
int stub_all_idle() {
    run_queues();
    for (auto &kv : g_queue)
        if (!kv.second.empty()) return 0;
    return 1;
}
void stub_capture(void *s, int on) {
    if (on) g_caller_capture.insert((hipStream_t)s);
    else g_caller_capture.erase((hipStream_t)s);
}
void stub_fail(const char *name, int nth) {
    if (nth > 0) g_fail[name] = nth;
    else g_fail.erase(name);
}
void stub_stay(int bin, int orientations) { g_stay[bin] = orientations; }
long long stub_allocs() { return (long long)g_allocs; }
}

// ---------------------------------------------------------------------------
// Kernel launchers
namespace dockgpu {
size_t dock_lds_bytes(int nmax, int waves) { return (size_t)nmax * 64 + (size_t)waves * (nmax * 48 + 2048); }
size_t select_lds_bytes(int, int, int, int, int) { return 1024; }
int select_sel_lds(int nmax, int waves, int, int K) { return (waves + K) * nmax * 12 <= 160 * 1024; }
size_t falign_lds_bytes(int, int, int) { return 1024; }
size_t align_lds_min(int, int, int) { return 1024; }
size_t plain_lds_bytes(int, int) { return 1024; }
int dock_blocks_per_cu(int, int, int) { return 4; }
int select_blocks_per_cu(int, int, int, int) { return 2; }
int falign_blocks_per_cu(int, int) { return 8; }
int align_blocks_per_cu(int, int, int, int) { return 1; }
int align_bound_blocks_per_cu(int) { return 4; }
hipError_t launch_build_cubes(const float *, float4 *, int, int, int, int, hipStream_t s) { return launched("cubes", s); }
hipError_t launch_reset(int *counters, int first, int count, hipStream_t s) {
    std::fill(counters + first, counters + first + count, 0);
    return launched(text("reset first=", first, " count=", count), s);
}
hipError_t launch_prep(const GridArgs &, const SearchArgs &sa, const LibArgs &la, const WorkArgs &ws, const OutArgs &, hipStream_t s) {
    for (int l = 0; l < la.L; ++l) {
        const int bin = (la.atom_off[l + 1] - la.atom_off[l] - 1) >> 5;
        ws.counters[sa.groups > 1 ? bin * sa.groups : l / ws.chunk * kNumBins + bin] += 1;
    }
    return launched(text("prep chunk=", ws.chunk), s);
}
hipError_t launch_prep_one(const GridArgs &, const SearchArgs &, const LibArgs &, const WorkArgs &, const OutArgs &, int l, hipStream_t s) { return launched(text("prep_one l=", l), s); }
hipError_t launch_atlas_count(const GridArgs &, int4 *, hipStream_t s) { return launched("atlas_count", s); }
hipError_t launch_atlas_fill(const GridArgs &, int4 *, const int *, float4 *, int, hipStream_t s) { return launched("atlas_fill", s); }
hipError_t launch_value_range(const float *, long long, uint32_t *, hipStream_t s) { return launched("value_range", s); }
hipError_t launch_bounds(const GridArgs &, const BoundArgs &, const float *, const uint32_t *, unsigned short *, hipStream_t s) { return launched("bounds", s); }
hipError_t launch_bound_probe(const GridArgs &, const BoundArgs &, const uint32_t *, int *stay, hipStream_t s) {
    for (int b = 0; b < kNumBins; ++b) stay[b] = g_stay[b] * kBoundProbes;
    return launched("bound_probe", s);
}
hipError_t launch_align(int bin, int lst, int blocks, int, const GridArgs &, const SearchArgs &, const LibArgs &, const WorkArgs &, hipStream_t s) { return launched(text("align bin=", bin, " lst=", lst, " blocks=", blocks), s); }
hipError_t launch_align_bound(int bin, int lst, int blocks, const GridArgs &, const SearchArgs &, const LibArgs &, const WorkArgs &, const BoundArgs &, hipStream_t s) { return launched(text("align_bound bin=", bin, " lst=", lst, " blocks=", blocks), s); }
hipError_t launch_dock(int bin, int lst, int blocks, int waves, const GridArgs &, const SearchArgs &, const LibArgs &, const WorkArgs &, hipStream_t s) { return launched(text("dock bin=", bin, " lst=", lst, " blocks=", blocks, " waves=", waves), s); }
hipError_t launch_select(int bin, int lst, int blocks, int waves, const GridArgs &, const SearchArgs &, const LibArgs &, const WorkArgs &, const OutArgs &, int, hipStream_t s) { return launched(text("select bin=", bin, " lst=", lst, " blocks=", blocks, " waves=", waves), s); }
hipError_t launch_falign(int bin, int lst, int blocks, int waves, const GridArgs &, const SearchArgs &, const LibArgs &, const WorkArgs &, const OutArgs &, int, int xcds, hipStream_t s) { return launched(text("falign bin=", bin, " lst=", lst, " blocks=", blocks, " waves=", waves, " xcds=", xcds), s); }
hipError_t launch_out(int bin, int lst, int blocks, const SearchArgs &, const LibArgs &, const WorkArgs &, const OutArgs &, int, hipStream_t s) { return launched(text("out bin=", bin, " lst=", lst, " blocks=", blocks), s); }
hipError_t launch_rescore(const ContactArgs &, const SearchArgs &, const LibArgs &, const OutArgs &, int, int blocks, hipStream_t s) { return launched(text("rescore blocks=", blocks), s); }
hipError_t launch_plain(int l, int, int, const GridArgs &, const SearchArgs &, const LibArgs &, const WorkArgs &, const OutArgs &, hipStream_t s) { return launched(text("plain l=", l), s); }
}  // namespace dockgpu
