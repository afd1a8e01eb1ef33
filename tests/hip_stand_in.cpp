// CPU stand-in for the parts of the HIP runtime that the library's host code calls, for sanitizer
// runs of that code (assembly, solves, serving) without a device: memory comes from the heap,
// streams, events and graphs are heap objects, launches do nothing except the two kernels whose
// results the solver's host part reads.  It aborts on what the runtime's documentation forbids:
//   - work on the legacy stream while a blocking stream is being captured (by any thread); it also
//     counts both, as the two meet only now and then,
//   - allocation, release, synchronisation or a memory fill in a thread that captures,
//   - release of memory that is not allocated, launches outside the device's limits.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

namespace {

struct Stream {
    bool blocking = true;
    bool captured = false;            // part of a capture under way
    std::vector<Stream *> joined;     // origin of a capture: the streams that joined it
    Stream *origin = nullptr;
    int touched = 0;
};
struct Event {
    Stream *origin = nullptr;         // recorded inside the capture that began on this stream
};
struct Graph {
    int alive = 1;
};

std::mutex g_mu;
std::map<const void *, std::string> g_names;
std::set<void *> g_live;
int g_blocking_captured = 0;
long g_legacy = 0, g_blocking = 0;
std::atomic<long> g_launches{0}, g_graphs{0};
thread_local bool t_capturing = false;
thread_local dim3 t_grid, t_block;
thread_local size_t t_shm;
thread_local hipStream_t t_stream;

[[noreturn]] void die(const char *what)
{
    std::fprintf(stderr, "stand-in: %s\n", what);
    std::abort();
}
void not_capturing(const char *what)
{
    if (t_capturing) die(what);
}
Stream *str(hipStream_t s) { return reinterpret_cast<Stream *>(s); }
Event *evt(hipEvent_t e) { return reinterpret_cast<Event *>(e); }
// work on stream s, on the legacy stream where it is null
void work_on(hipStream_t s)
{
    if (std::rand() % 16 == 0) std::this_thread::yield();
    std::lock_guard<std::mutex> lk(g_mu);
    if (s) {
        str(s)->touched++;
        return;
    }
    ++g_legacy;
    if (g_blocking_captured > 0) die("legacy stream used while a blocking stream is captured");
}
void join_capture(Stream *s, Stream *origin)   // g_mu held
{
    if (s->captured) return;
    s->captured = true;
    s->origin = origin;
    if (s != origin) origin->joined.push_back(s);
    if (s->blocking) {
        ++g_blocking_captured;
        ++g_blocking;
    }
}
void leave_capture(Stream *s)
{
    if (s->blocking) --g_blocking_captured;
    s->captured = false;
    s->origin = nullptr;
}

}  // namespace

extern "C" {

hipError_t hipMalloc(void **p, size_t n)
{
    not_capturing("allocation while capturing");
    *p = std::calloc(1, n);
    std::lock_guard<std::mutex> lk(g_mu);
    g_live.insert(*p);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p)
{
    not_capturing("release while capturing");
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (p && !g_live.erase(p)) die("release of memory that is not allocated");
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    not_capturing("synchronous copy while capturing");
    work_on(nullptr);
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    work_on(st);
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st)
{
    not_capturing("memory fill in a capture");
    work_on(st);
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *f, size_t *t)
{
    *f = *t = (size_t)200 << 30;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *d)
{
    *d = 1;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned flags)
{
    auto *n = new Stream();
    n->blocking = !(flags & hipStreamNonBlocking);
    *s = reinterpret_cast<hipStream_t>(n);
    return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t *s) { return hipStreamCreateWithFlags(s, hipStreamDefault); }
hipError_t hipStreamDestroy(hipStream_t s)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (str(s)->captured) die("stream destroyed while it is captured");
    }
    delete str(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    not_capturing("synchronisation while capturing");
    work_on(s);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = reinterpret_cast<hipEvent_t>(new Event());
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete evt(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    work_on(s);
    std::lock_guard<std::mutex> lk(g_mu);
    evt(e)->origin = str(s)->captured ? str(s)->origin : nullptr;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    work_on(s);
    std::lock_guard<std::mutex> lk(g_mu);
    if (evt(e)->origin) join_capture(str(s), evt(e)->origin);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    not_capturing("synchronisation while capturing");
    std::lock_guard<std::mutex> lk(g_mu);
    if (evt(e)->origin) die("wait for an event of a capture");
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t)
{
    *t = 1.0f;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c)
{
    std::lock_guard<std::mutex> lk(g_mu);
    *c = str(s)->captured ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    std::lock_guard<std::mutex> lk(g_mu);
    t_capturing = true;
    join_capture(str(s), str(s));
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g)
{
    std::this_thread::sleep_for(std::chrono::milliseconds(2));   // the other threads come to see the capture
    std::lock_guard<std::mutex> lk(g_mu);
    if (str(s)->origin != str(s)) die("end of a capture that did not begin here");
    for (Stream *j : str(s)->joined) leave_capture(j);
    str(s)->joined.clear();
    leave_capture(str(s));
    t_capturing = false;
    *g = reinterpret_cast<hipGraph_t>(new Graph());
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    if (!reinterpret_cast<Graph *>(g)->alive) die("graph is gone");
    *e = reinterpret_cast<hipGraphExec_t>(new Graph());
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete reinterpret_cast<Graph *>(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t g)
{
    delete reinterpret_cast<Graph *>(g);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t g, hipStream_t s)
{
    g_graphs++;
    if (!reinterpret_cast<Graph *>(g)->alive) die("graph is gone");
    work_on(s);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static double fixed[16];
    *p = fixed;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *)
{
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    std::lock_guard<std::mutex> lk(g_mu);
    g_names[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s)
{
    t_grid = g;
    t_block = b;
    t_shm = m;
    t_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s)
{
    *g = t_grid;
    *b = t_block;
    *m = t_shm;
    *s = t_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t shm, hipStream_t s)
{
    g_launches++;
    work_on(s);
    const size_t threads = (size_t)b.x * b.y * b.z;
    if (!g.x || !g.y || !g.z || g.y > 65535 || g.z > 65535 || threads < 1 || threads > 1024 || shm > 163840)
        die("launch outside the limits");
    std::string n;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        n = g_names[f];
    }
    if (n.find("k_norm2_b") != std::string::npos) {   // (n, x, out): norms of 1
        double *out = *static_cast<double **>(args[2]);
        for (unsigned c = 0; c < g.x; ++c) out[c] = 1.0;
    } else if (n.find("k_gs_fin") != std::string::npos) {   // a column of coefficients, |y| = 0.4
        const int r = *static_cast<int *>(args[1]), k = *static_cast<int *>(args[7]);
        const int *run = *static_cast<const int **>(args[5]);
        double *out = *static_cast<double **>(args[15]);
        for (int c = 0; c < r; ++c)
            for (int i = 0; run[c] && i <= k; ++i) {
                out[2 * ((size_t)c * (k + 1) + i)] = i == k ? 0.4 : (i == k - 1 ? 1.0 : 0.05);
                out[2 * ((size_t)c * (k + 1) + i) + 1] = 0.0;
            }
    }
    return hipSuccess;
}

}  // extern "C"

__attribute__((destructor)) static void report()
{
    std::fprintf(stderr, "stand-in: %ld launches, %ld graph launches, %ld operations on the legacy stream, %ld blocking streams "
                         "captured, %zu allocations left\n", g_launches.load(), g_graphs.load(), g_legacy, g_blocking, g_live.size());
}
