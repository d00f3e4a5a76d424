// A stand-in for the HIP runtime that runs nothing: device memory is address
// space that nobody touches, copies do nothing, and every kernel launch is
// recorded (kernel, grid, block).  Loaded ahead of liblbm.so in a process of
// its own, it shows on the CPU which kernels a call enqueues and what the call
// returns when the runtime refuses something.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <map>
#include <system_error>
#include <vector>

namespace {
struct Launch {
    const void *fn;
    dim3 grid, block;
};
std::vector<Launch> launches;
std::map<void *, size_t> blocks;
hipError_t last = hipSuccess;
long events = 0;  // alive
long refuse_launch = -1;  // launches until one is refused; -1: never
int refuse_pinned = 0, refuse_threads = 0, refuse_device = 0;
char device_symbol[256];

hipError_t set(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}

hipError_t take(void **p, size_t n)
{
    *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    blocks[*p] = n;
    return hipSuccess;
}

hipError_t give(void *p)
{
    if (p) munmap(p, blocks[p]);
    blocks.erase(p);
    return hipSuccess;
}
}  // namespace

extern "C" {
long rec_count() { return (long)launches.size(); }
void rec_clear() { launches.clear(); }
const char *rec_name(long i)
{
    Dl_info d{};
    return dladdr(launches[i].fn, &d) && d.dli_sname ? d.dli_sname : "?";
}
unsigned rec_grid(long i, int axis) { return axis == 0 ? launches[i].grid.x : launches[i].grid.y; }
unsigned rec_block(long i, int axis) { return axis == 0 ? launches[i].block.x : launches[i].block.y; }
long rec_blocks() { return (long)blocks.size(); }  // allocations alive
long rec_events() { return events; }
void rec_refuse(long launch, int pinned, int threads, int device)
{
    refuse_launch = launch;
    refuse_pinned = pinned;
    refuse_threads = threads;
    refuse_device = device;
}

hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t *p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950:recorded");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 163840, hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { return refuse_device ? set(hipErrorOutOfMemory) : take(p, n); }
hipError_t hipFree(void *p) { return give(p); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return refuse_pinned ? set(hipErrorOutOfMemory) : take(p, n); }
hipError_t hipHostFree(void *p) { return give(p); }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = device_symbol, hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError()
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "recorded error"; }
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
};
static Config config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    config = {g, b, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    *g = config.grid;
    *b = config.block;
    *lds = config.lds;
    *s = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **, size_t, hipStream_t)
{
    if (refuse_launch >= 0 && refuse_launch-- == 0) return set(hipErrorInvalidConfiguration);
    if (grid.y > 65535 || (unsigned long long)grid.x * block.x > 0xffffffffull) return set(hipErrorInvalidConfiguration);
    launches.push_back({fn, grid, block});
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)malloc(8), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return free(s), hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return *g = (hipGraph_t)malloc(8), hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    return *x = (hipGraphExec_t)malloc(8), hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return free(g), hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return free(x), hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)malloc(8), ++events, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return free(e), --events, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }

// std::thread's start, in place of the C++ library's.
void _ZNSt6thread15_M_start_threadESt10unique_ptrINS_6_StateESt14default_deleteIS1_EEPFvvE(void *self, void *state,
                                                                                         void (*depend)())
{
    if (refuse_threads) throw std::system_error(EAGAIN, std::generic_category());
    using Start = void (*)(void *, void *, void (*)());
    static const Start next = (Start)dlsym(
        RTLD_NEXT, "_ZNSt6thread15_M_start_threadESt10unique_ptrINS_6_StateESt14default_deleteIS1_EEPFvvE");
    next(self, state, depend);
}
}
