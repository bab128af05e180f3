// fake_hip.h -- a stand-in for the HIP runtime, for tests of the library's host side on
// the CPU: two devices, streams and events that belong to one of them, device memory
// that is the host's, and counted host allocations. As HIP does, an event is recorded
// only on a stream of its own device. Kernels are counted, not run; nothing is captured.
// Included by one source file of a program.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

struct ihipStream_t {
    int dev;
};
struct ihipEvent_t {
    int dev;
};

namespace fake {
bool no_pinned = false;   // pinned host memory is used up
int current = 0, launches = 0, host_allocs = 0, host_frees = 0, events = 0, copies = 0, dev_allocs = 0;
hipError_t last = hipSuccess;
hipError_t note(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}
}  // namespace fake

extern "C" {
char __hip_fatbin[16];
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* s)
{
    *g = *b = dim3(1);
    *n = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t)
{
    fake::launches += 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d)
{
    *d = fake::current;
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    if (d < 0 || d > 1) return fake::note(hipErrorInvalidDevice);
    fake::current = d;
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d)
{
    *d = s ? s->dev : fake::current;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    if (fake::no_pinned) return fake::note(hipErrorOutOfMemory);
    *p = std::malloc(n);
    fake::host_allocs += 1;
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    std::free(p);
    fake::host_frees += 1;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    *e = new ihipEvent_t{fake::current};
    fake::events += 1;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete e;
    fake::events -= 1;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    return e->dev == (s ? s->dev : fake::current) ? hipSuccess : fake::note(hipErrorInvalidHandle);
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetLastError()
{
    const hipError_t e = fake::last;
    fake::last = hipSuccess;
    return e;
}
hipError_t hipMemcpy2DAsync(void* dst, size_t dp, const void* src, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t)
{
    for (size_t r = 0; r < h; ++r)
        std::memcpy(static_cast<char*>(dst) + r * dp, static_cast<const char*>(src) + r * sp, w);
    fake::copies += 1;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n)
{
    fake::dev_allocs += 1;
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    return *p ? hipSuccess : fake::note(hipErrorOutOfMemory);
}
hipError_t hipFree(void* p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* dst, int v, size_t n, hipStream_t)
{
    std::memset(dst, v, n);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = new ihipStream_t{fake::current};
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    delete s;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    static std::vector<char> array(size_t(4) << 20);
    *p = array.data();
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return fake::note(hipErrorNotSupported); }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return fake::note(hipErrorNotSupported); }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    return fake::note(hipErrorNotSupported);
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return fake::note(hipErrorNotSupported); }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

#define CHECK(x)                                                       \
    do {                                                               \
        if (!(x)) {                                                    \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);        \
            return 1;                                                  \
        }                                                              \
    } while (0)
