#include "fake_hip.h"

#include <cstdlib>
#include <cstring>

namespace fake {

// (built on first use: the library registers its kernels before this file's constructors run)
Device& device()
{
    static Device* d = new Device();
    return *d;
}
static std::map<const void*, std::string>& kernels()
{
    static auto* m = new std::map<const void*, std::string>();
    return *m;
}

bool fails()
{
    Device& d = device();
    if (d.calls++ != d.fail_at) return false;
    d.failed = true;
    return true;
}

static hipError_t work(hipStream_t s)
{
    if (fails()) return hipErrorUnknown;
    device().pending.insert(s);
    return hipSuccess;
}

static dim3 g_grid, g_block;

}  // namespace fake

using namespace fake;

extern "C" {

void** __hipRegisterFatBinary(const void*)
{
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    kernels()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t s)
{
    g_grid = grid;
    g_block = block;
    device().pending.insert(s);
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s)
{
    *grid = g_grid;
    *block = g_block;
    *shared = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t)
{
    device().launches.push_back({kernels()[f], grid.x, block.x});
    return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n)
{
    Device& d = device();
    *p = nullptr;
    if (fails()) return hipErrorUnknown;
    if (n > d.capacity - d.used) return hipErrorOutOfMemory;
    d.live[d.next] = n;
    *p = d.next;
    d.next += (n + 4095) / 4096 * 4096;
    d.used += n;
    if (d.used > d.peak) d.peak = d.used;
    return hipSuccess;
}
// waits for the device, as the runtime's does
hipError_t hipFree(void* p)
{
    Device& d = device();
    auto i = d.live.find((char*)p);
    if (i == d.live.end()) return hipErrorInvalidValue;
    d.freed.push_back(i->second);
    d.used -= i->second;
    d.live.erase(i);
    d.pending.clear();
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    if (fails()) return hipErrorUnknown;
    *p = calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free_b, size_t* total)
{
    *free_b = device().capacity - device().used;
    *total = device().capacity;
    return hipSuccess;
}
hipError_t hipDeviceTotalMem(size_t* n, hipDevice_t)
{
    *n = device().capacity;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int)
{
    *v = 256;  // compute units: the only one asked for
    return hipSuccess;
}
// Workgroups per compute unit as registers and LDS allow them on gfx950
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t)
{
    const std::string& k = kernels()[f];
    *n = 2;
    if (k.find("k3_march") != std::string::npos)
        *n = block != 256 || k.find("k3_marchIff") == std::string::npos ? 1 : (k.find("Li19E") != std::string::npos ? 3 : 2);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    *p = (void*)((size_t)1 << 39);
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetLastError(void) { return fails() ? hipErrorUnknown : hipSuccess; }

hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return fails() ? hipErrorUnknown : hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t s) { return work(s); }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t s) { return work(s); }
hipError_t hipStreamSynchronize(hipStream_t s)
{
    device().pending.erase(s);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    if (fails()) return hipErrorUnknown;
    *s = (hipStream_t)(device().next += 64);
    device().streams.insert(*s);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    device().streams.erase(s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return fails() ? hipErrorUnknown : hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    if (fails()) return hipErrorUnknown;
    *e = (hipEvent_t)(device().next += 64);
    device().events.insert(*e);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    device().events.erase(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return fails() ? hipErrorUnknown : hipSuccess; }

hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    *g = (hipGraph_t)1;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    *e = (hipGraphExec_t)1;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s)
{
    device().pending.insert(s);
    return hipSuccess;
}

}  // extern "C"
