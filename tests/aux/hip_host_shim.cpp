// Stand-ins for the HIP runtime calls of the library's host code, so that its launch
// rules and its reads run on a machine without a GPU: "device" memory is host memory,
// streams are synchronous, and a kernel's launch does nothing. Loaded with global symbols
// before libgs.so.
#include <hip/hip_runtime_api.h>

#include <stdlib.h>
#include <string.h>
#include <xmmintrin.h>

#include <atomic>
#include <vector>

static int g_cus = 256, g_lanes = 1024; // compute units; lanes that one of them holds
static const void *g_known;              // memory of the runtime's own
static struct { dim3 grid, block; size_t lds; hipStream_t st; } g_call; // (of the one thread that launches)
static hipError_t g_error = hipSuccess;
static std::atomic<int> g_pinned{0}, g_events{0};
static std::vector<unsigned> g_grids; // workgroups of each launch

extern "C" {

void shim_device(int cus, int lanes) { g_cus = cus, g_lanes = lanes; }
void shim_known(const void *p) { g_known = p; }
int shim_pinned() { return g_pinned; } // pinned allocations alive
int shim_events() { return g_events; } // events alive
int shim_launches() { return (int)g_grids.size(); }
unsigned shim_grid(int i) { return g_grids[i]; }
// Denormals are zero and flushed to zero in the calling thread (and those it starts).
void shim_flush_denormals(int on) { _mm_setcsr(on ? _mm_getcsr() | 0x8040 : _mm_getcsr() & ~0x8040u); }

hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    if (a != hipDeviceAttributeMultiprocessorCount) return hipErrorInvalidValue;
    return *v = g_cus, hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int block, size_t)
{
    return *n = g_lanes >= block ? g_lanes / block : 1, hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) { return *d = 0, hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    return *p ? ++g_pinned, hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p)
{
    free(p);
    return --g_pinned, hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = (hipEvent_t)malloc(1);
    return ++g_events, hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    free(e);
    return --g_events, hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    if (p != g_known) return hipErrorInvalidValue;
    return a->type = hipMemoryTypeDevice, hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st)
{
    g_call = {grid, block, lds, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st)
{
    *grid = g_call.grid, *block = g_call.block, *lds = g_call.lds, *st = g_call.st;
    return hipSuccess;
}
// The runtime's limit: less than 2^32 threads in a dimension of the grid.
hipError_t hipLaunchKernel(const void *, dim3 grid, dim3 block, void **, size_t, hipStream_t)
{
    g_grids.push_back(grid.x);
    return g_error = (double)grid.x * block.x < 4294967296.0 ? hipSuccess : hipErrorInvalidConfiguration;
}
hipError_t hipGetLastError()
{
    const hipError_t e = g_error;
    return g_error = hipSuccess, e;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
}
