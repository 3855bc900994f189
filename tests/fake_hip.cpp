// A stand-in for the HIP runtime, to run the host side of the library without
// a GPU: device memory is host memory, kernels do nothing, streams complete
// when they are synchronised.  It counts what tests ask about (fake_count) and
// can refuse host allocations of the calling thread (fake_refuse_new).
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <unistd.h>
#include <utility>
#include <vector>

#include "../paper_2311_11348_amd/csrc/swe_internal.h"

namespace {

typedef std::set<std::pair<void *, long>> Waits;   // (stream, launches issued on it)
struct Stream { long issued = 0, done = 0; Waits waits; };

std::mutex mx;
std::map<void *, Stream> streams;
std::map<void *, Waits> events;                    // what an event was recorded after
std::map<void *, Waits> execs;                     // launches of a graph
std::map<std::string, long> counts;
std::map<void *, size_t> sizes;
std::atomic<int> in_graph_call{0};
thread_local bool refuse = false;
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;

// held while the maps above are used, whose own allocations are not refused
struct Model {
    std::lock_guard<std::mutex> lock{mx};
    const bool was = refuse;
    Model() { refuse = false; }
    ~Model() { refuse = was; }
};

void done(void *s, long n)
{
    Stream &t = streams[s];
    if (n > t.done) t.done = n;
    for (const auto &w : Waits(t.waits))
        if (streams[w.first].done < w.second) done(w.first, w.second);
}

// building and destroying graphs: how many calls at once
struct GraphCall {
    GraphCall()
    {
        const int n = ++in_graph_call;
        Model l;
        if (n > counts["graph calls at once"]) counts["graph calls at once"] = n;
    }
    ~GraphCall()
    {
        usleep(300);
        --in_graph_call;
    }
};

// an allocation, a free, a stream made or ended: whether a graph is being built or destroyed meanwhile
struct OtherCall {
    OtherCall() { look(); }
    ~OtherCall()
    {
        usleep(20);
        look();
    }
    static void look()
    {
        if (in_graph_call.load() == 0) return;
        Model l;
        counts["other calls beside graph calls"] += 1;
    }
};

hipError_t alloc(void **p, size_t n)
{
    OtherCall call;
    *p = calloc(1, n ? n : 1);
    Model l;
    sizes[*p] = n;
    counts["bytes"] += (long)n;
    if (mode != hipStreamCaptureModeRelaxed) counts["allocations a capture elsewhere forbids"] += 1;
    return hipSuccess;
}

hipError_t release(void *p)
{
    OtherCall call;
    {
        Model l;
        counts["bytes"] -= (long)sizes[p];
        sizes.erase(p);
    }
    free(p);
    return hipSuccess;
}

template <typename T>
hipError_t handle(T *p)
{
    *p = (T)malloc(16);
    return hipSuccess;
}

}  // namespace

void *operator new(size_t n)
{
    void *p = refuse ? nullptr : malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(size_t n, const std::nothrow_t &) noexcept { return refuse ? nullptr : malloc(n ? n : 1); }
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

extern "C" {

long fake_count(const char *what)
{
    Model l;
    return counts[what];
}
void fake_refuse_new(int on) { refuse = on != 0; }

hipError_t hipMalloc(void **p, size_t n) { return alloc(p, n); }
hipError_t hipFree(void *p) { return release(p); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags)
{
    OtherCall call;
    Model l;
    counts["pinned allocations"] += 1;
    if (mode != hipStreamCaptureModeRelaxed) counts["allocations a capture elsewhere forbids"] += 1;
    if (!(flags & hipHostMallocCoherent)) counts["pinned allocations not coherent"] += 1;
    *p = calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    OtherCall call;
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t)
{
    for (size_t i = 0; i < h; ++i) memcpy((char *)d + i * dp, (const char *)s + i * sp, w);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    OtherCall call;
    return handle(s);
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    OtherCall call;
    free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    Model l;
    done(s, streams[s].issued);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st)
{
    *st = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m)
{
    std::swap(mode, *m);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    Model l;
    for (const auto &w : events[e]) streams[s].waits.insert(w);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return handle(e); }
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    Model l;
    events[e] = Waits{{s, streams[s].issued}};
    for (const auto &w : streams[s].waits) events[e].insert(w);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    Model l;
    for (const auto &w : Waits(events[e])) done(w.first, w.second);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *f, hipEvent_t, hipEvent_t)
{
    *f = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipGetDeviceCount(int *v)
{
    *v = 1;
    return hipSuccess;
}
hipError_t hipGraphCreate(hipGraph_t *g, unsigned)
{
    GraphCall call;
    return handle(g);
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    GraphCall call;
    free(g);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    GraphCall call;
    handle(x);
    Model l;
    counts["graphs built"] += 1;
    execs[*x].clear();
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    GraphCall call;
    Model l;
    for (const auto &w : execs[x])
        if (streams[w.first].done < w.second) counts["graphs destroyed in flight"] += 1;
    execs.erase(x);
    free(x);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s)
{
    Model l;
    execs[x].insert({s, ++streams[s].issued});
    return hipSuccess;
}

}  // extern "C"

namespace swe {

hipError_t launch_build_tiles(const MeshView &, int, const TileView &, int *, hipStream_t)
{
    Model l;
    counts["tile builds"] += 1;
    return hipSuccess;
}
bool stage_sh_supported(int p, bool) { return p >= 1; }
hipError_t launch_step_sh(int, bool, const void *, const TileView &, double, int, Sink &)
{
    Model l;
    counts["one-launch steps"] += 1;
    return hipSuccess;
}

}  // namespace swe
