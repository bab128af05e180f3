// readback_host.cc -- the host side of csrc/lbvp_readback.hip on a stand-in for the HIP
// runtime: two devices, streams and events that belong to one of them, and counted
// host allocations. As HIP does, an event is recorded only on a stream of its own device.
// Kernels are counted, not run. usage: readback_host CHECK; exits with 0 if it holds.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "lbvp_readback.h"

struct ihipStream_t {
    int dev;
};
struct ihipEvent_t {
    int dev;
};

namespace fake {
bool no_pinned = false;   // pinned host memory is used up
int current = 0, launches = 0, host_allocs = 0, host_frees = 0, events = 0, copies = 0;
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
}

#define CHECK(x)                                                       \
    do {                                                               \
        if (!(x)) {                                                    \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);        \
            return 1;                                                  \
        }                                                              \
    } while (0)

constexpr int NX = 1500, ROWS = 1500, PITCH = 1536;   // three staging buffers of floats a plane

static hipError_t read_some(hipStream_t s, const std::vector<float>& dev, std::vector<double>& out)
{
    const int64_t off[2] = {0, (int64_t)ROWS * PITCH};
    out.assign(2 * (size_t)NX * ROWS, -1.0);
    double* dst[2] = {out.data(), out.data() + (size_t)NX * ROWS};
    return lbvp::read_planes(s, false, dev.data(), off, 2, PITCH, NX, ROWS, dst);
}

// Streams of either device, whichever is current: the staging belongs to the stream's
// device and the caller's current device stays as it was.
static int devices()
{
    ihipStream_t on0{0}, on1{1};
    std::vector<float> dev(2 * (size_t)ROWS * PITCH, 1.0f);
    std::vector<uint8_t> mask((size_t)NX * ROWS, 1), dmask((size_t)PITCH * ROWS, 0);
    std::vector<double> out;
    lbvp::ReadbackUser user;
    for (int k = 0; k < 8; ++k) {
        fake::current = k & 1;
        ihipStream_t* s = k & 2 ? &on1 : &on0;
        CHECK(lbvp::write_mask(s, dmask.data(), PITCH, NX, ROWS, mask.data()) == hipSuccess);
        CHECK(read_some(s, dev, out) == hipSuccess);
        CHECK(fake::current == (k & 1));
        CHECK(read_some(nullptr, dev, out) == hipSuccess);
    }
    CHECK(fake::host_allocs == 4);   // a pair per device, used again
    CHECK(fake::launches > 0);
    return 0;
}

// Without pinned memory the calls copy through pageable memory, leave no error behind,
// and use staging again when there is some.
static int pageable()
{
    ihipStream_t s{0};
    std::vector<float> dev(2 * (size_t)ROWS * PITCH);
    for (size_t k = 0; k < dev.size(); ++k) dev[k] = (float)(k % 8191);
    std::vector<uint8_t> mask((size_t)NX * ROWS), dmask((size_t)PITCH * ROWS, 255);
    for (size_t k = 0; k < mask.size(); ++k) mask[k] = (uint8_t)(k % 251);
    std::vector<double> out;
    lbvp::ReadbackUser user;
    fake::no_pinned = true;
    CHECK(lbvp::write_mask(&s, dmask.data(), PITCH, NX, ROWS, mask.data()) == hipSuccess);
    CHECK(read_some(&s, dev, out) == hipSuccess);
    CHECK(hipGetLastError() == hipSuccess);
    CHECK(fake::launches == 0 && fake::host_allocs == fake::host_frees);
    for (int r = 0; r < ROWS; ++r)
        for (int i = 0; i < PITCH; ++i) {
            CHECK(dmask[(size_t)r * PITCH + i] == (i < NX ? mask[(size_t)r * NX + i] : 255));
            for (int q = 0; q < 2 && i < NX; ++q)
                CHECK(out[((size_t)q * ROWS + r) * NX + i] == dev[((size_t)q * ROWS + r) * PITCH + i]);
        }
    fake::no_pinned = false;
    CHECK(read_some(&s, dev, out) == hipSuccess);
    CHECK(fake::launches > 0);
    return 0;
}

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "devices")) return devices();
    if (!std::strcmp(what, "pageable")) return pageable();
    std::printf("unknown check %s\n", what);
    return 2;
}
