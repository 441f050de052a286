// A HIP runtime that launches nothing and writes down what it was asked to
// launch: the library's host code, linked against it, runs on a machine
// without a GPU and shows which kernels it chose, how it cut the lattice and
// which buffer each launch reads and writes.  Device memory is host memory.
#include <hip/hip_runtime.h>

#include <condition_variable>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "plbm_sweep.h"

namespace {

struct Launch {
    std::string name;
    unsigned grid, block;
    size_t lds;
    void *src, *dst;               // the first two arguments
    int extra[7];                  // those that place the work (see hipLaunchKernel)
};

std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> k;
    return k;
}
std::vector<Launch> launches;
long long bytes_held = 0, mallocs_left = -1;
std::mutex mu;                     // of what follows and of the launches
std::condition_variable changed;
hipStream_t busy = nullptr;        // a stream whose synchronisation waits
bool waiting = false;              // somebody does
struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t st;
} config;

void *take(size_t n)
{
    if (mallocs_left == 0) return nullptr;
    if (mallocs_left > 0) --mallocs_left;
    auto *p = static_cast<size_t *>(std::malloc(n + 64));
    if (!p) return nullptr;
    *p = n;
    bytes_held += (long long)n;
    return p + 8;
}
void give(void *q)
{
    if (!q) return;
    size_t *p = static_cast<size_t *>(q) - 8;
    bytes_held -= (long long)*p;
    std::free(p);
}

} // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *)
{
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    kernels()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st)
{
    config = {grid, block, lds, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st)
{
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *st = config.st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t)
{
    Launch l{kernels()[f], grid.x * grid.y * grid.z, block.x, lds, *(void **)args[0], *(void **)args[1], {}};
    auto is = [&](const char *s) { return l.name.find(s) != std::string::npos; };
    if (is("k_tube"))                                           // tile, reach, steps
        for (int k = 0; k < 3; ++k) l.extra[k] = *(int *)args[3 + k];
    else if (is("k_step2d_sweep") || is("k_sweep_q9") || is("k_pair_gen"))
        std::memcpy(l.extra, args[3], sizeof(SweepGrid));
    std::lock_guard<std::mutex> lock(mu);
    launches.push_back(l);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return (*p = take(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return hipMalloc(p, n); }
hipError_t hipFree(void *p)
{
    give(p);
    return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memset(d, 0, n);          // sums of zero: nothing ran
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static double scratch[2 * (8192 + 1) * 4];
    *p = scratch;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t st)
{
    std::unique_lock<std::mutex> lock(mu);
    if (busy && st == busy) {
        waiting = true;
        changed.notify_all();
        changed.wait(lock, [] { return !busy; });
        waiting = false;
    }
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    *g = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *e = reinterpret_cast<hipGraphExec_t>(&config);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }

// What was recorded.
void rec_clear() { launches.clear(); }
int rec_count() { return (int)launches.size(); }
const char *rec_name(int i) { return launches[i].name.c_str(); }
void rec_launch(int i, unsigned *grid, unsigned *block, size_t *lds, void **src, void **dst, int *extra)
{
    const Launch &l = launches[i];
    *grid = l.grid;
    *block = l.block;
    *lds = l.lds;
    *src = l.src;
    *dst = l.dst;
    std::memcpy(extra, l.extra, sizeof(l.extra));
}
// Work on the stream st does not end until rec_busy(0); rec_await returns once a
// call waits for it.
void rec_busy(void *st)
{
    std::lock_guard<std::mutex> lock(mu);
    busy = static_cast<hipStream_t>(st);
    changed.notify_all();
}
void rec_await()
{
    std::unique_lock<std::mutex> lock(mu);
    changed.wait(lock, [] { return waiting; });
}
// Device memory in use, and how many more allocations succeed (-1: all).
long long rec_bytes() { return bytes_held; }
void rec_allow_mallocs(long long n) { mallocs_left = n; }
// The kernel's own placement of a thread in a strip (plbm_sweep.h).
int rec_sweep_side(const int *grid, int thread, int threads)
{
    SweepGrid g;
    std::memcpy(&g, grid, sizeof(g));
    return sweep_side(g, thread, threads);
}
}
