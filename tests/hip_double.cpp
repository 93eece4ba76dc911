// A stand-in for the HIP runtime on the CPU: librr.so's host code runs on it
// unchanged (tests/test_host_runtime.py loads it with global visibility before
// the library).  Device memory is host memory of a settable size; kernels do
// not run, their launches are logged; streams finish work only when something
// waits for it, so an object destroyed or freed too early is seen.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Graph {
    std::vector<std::string> work;
};
struct Exec {
    std::vector<std::string> work;
    long long last = 0;   // ticket of the last launch
};
struct Stream {
    bool capturing = false;   // by the library
    bool by_caller = false;   // by the caller (hd_set_capturing)
    hipStream_t origin = nullptr;
};
struct Event {
    long long ticket = 0;
    hipStream_t captured_on = nullptr;
};

std::map<const void *, std::string> g_kernels;
std::map<void *, size_t> g_mem;
std::map<hipStream_t, Stream> g_streams;
std::map<hipStream_t, Graph *> g_captures;   // by the capture's origin
std::string g_log, g_faults;
size_t g_used = 0, g_limit = (size_t)1 << 36;
long long g_ticket = 0, g_done = 0;          // work handed out, work known to be finished
int g_execs = 0, g_waits = 0;                // executable graphs alive; waits for the GPU
hipError_t g_last = hipSuccess;
dim3 g_grid, g_block;
size_t g_shmem = 0;
hipStream_t g_stream = nullptr;
char *g_symbol = nullptr;

hipError_t err(hipError_t e)
{
    if (e != hipSuccess) g_last = e;
    return e;
}

Graph *graph_of(hipStream_t s)
{
    Stream &st = g_streams[s];
    if (!st.capturing) return nullptr;
    auto it = g_captures.find(st.origin);
    return it == g_captures.end() ? nullptr : it->second;
}

void work(hipStream_t s, const std::string &text)
{
    if (Graph *g = graph_of(s)) {
        g->work.push_back(text);
        return;
    }
    if (g_streams[s].by_caller) g_log += "captured ";
    else ++g_ticket;
    g_log += text + "\n";
}

void not_in_capture(const char *what)
{
    for (auto &s : g_streams)
        if (s.second.by_caller) g_faults += std::string(what) + " during a capture\n";
}

}  // namespace

extern "C" {

// -- what the test reads and sets
const char *hd_log() { return g_log.c_str(); }
const char *hd_faults() { return g_faults.c_str(); }
int hd_last_error() { return (int)g_last; }
int hd_live_execs() { return g_execs; }
int hd_waits() { return g_waits; }
void hd_clear()
{
    g_log.clear();
    g_faults.clear();
}
void hd_set_memory(uint64_t bytes) { g_limit = bytes; }
uint64_t hd_used() { return g_used; }
void hd_set_capturing(uint64_t stream, int on) { g_streams[(hipStream_t)stream].by_caller = on != 0; }
uint64_t hd_buffer_end(uint64_t p)   // end of the allocation that p lies in, or 0
{
    auto it = g_mem.upper_bound((void *)p);
    if (it == g_mem.begin()) return 0;
    --it;
    const uint64_t end = (uint64_t)it->first + it->second;
    return p < end ? end : 0;
}

// -- code objects and launches
void **__hipRegisterFatBinary(const void *) { return (void **)&g_symbol; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    g_kernels[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s)
{
    g_grid = grid;
    g_block = block;
    g_shmem = shmem;
    g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *s)
{
    *grid = g_grid;
    *block = g_block;
    *shmem = g_shmem;
    *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t s)
{
    std::string t = g_kernels[f] + " grid " + std::to_string(grid.x) + " " + std::to_string(grid.y);
    if (g_kernels[f].find("k_vas_scan") != std::string::npos)   // (.., D) last of nine
        t += " D " + std::to_string((uint64_t) * (double **)args[8]);
    work(s, t);
    return hipSuccess;
}

// -- device and memory
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = p->maxSharedMemoryPerMultiProcessor = 160 << 10;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    not_in_capture("hipMalloc");
    *p = nullptr;
    if (g_used + n > g_limit) return err(hipErrorOutOfMemory);
    *p = calloc(1, n);
    if (!*p) return err(hipErrorOutOfMemory);
    g_mem[*p] = n;
    g_used += n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    g_done = g_ticket;   // waits for the device
    g_used -= g_mem[p];
    g_mem.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *avail, size_t *total)
{
    *avail = g_limit > g_used ? g_limit - g_used : 0;
    *total = g_limit;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    if (!g_symbol) g_symbol = (char *)calloc(1, (size_t)64 << 20);
    *p = g_symbol;
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    not_in_capture("hipMemcpy");
    g_done = g_ticket;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    memcpy(d, s, n);
    work(st, "copy");
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n)
{
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t s)
{
    memset(d, v, n);
    work(s, "memset");
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetLastError(void)
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}

// -- streams, events
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = (hipStream_t)malloc(16);
    g_streams[*s] = Stream();
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    g_streams.erase(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    not_in_capture("hipStreamSynchronize");
    ++g_waits;
    g_done = g_ticket;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void)
{
    ++g_waits;
    g_done = g_ticket;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = (hipEvent_t) new Event();
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete (Event *)e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    not_in_capture("hipEventRecord");
    ((Event *)e)->captured_on = g_streams[s].capturing ? g_streams[s].origin : nullptr;
    ((Event *)e)->ticket = g_ticket;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    ++g_waits;
    g_done = std::max(g_done, ((Event *)e)->ticket);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { return err(((Event *)e)->ticket <= g_done ? hipSuccess : hipErrorNotReady); }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.1f;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    if (hipStream_t o = ((Event *)e)->captured_on) {   // joins the capture
        g_streams[s].capturing = true;
        g_streams[s].origin = o;
    }
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st)
{
    *st = g_streams[s].by_caller || g_streams[s].capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}

// -- graphs
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    g_streams[s].capturing = true;
    g_streams[s].origin = s;
    g_captures[s] = new Graph();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g)
{
    for (auto &x : g_streams)
        if (x.second.origin == s) x.second = Stream();
    *g = (hipGraph_t)g_captures[s];
    g_captures.erase(s);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    Exec *e = new Exec();
    ++g_execs;
    e->work = ((Graph *)g)->work;
    *x = (hipGraphExec_t)e;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t)
{
    ((Exec *)x)->last = ++g_ticket;
    for (const std::string &t : ((Exec *)x)->work) g_log += "graph: " + t + "\n";
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    if (((Exec *)x)->last > g_done) g_faults += "executable graph destroyed before its launch has finished\n";
    --g_execs;
    delete (Exec *)x;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete (Graph *)g;
    return hipSuccess;
}
}
