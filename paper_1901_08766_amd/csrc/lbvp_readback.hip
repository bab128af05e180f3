// lbvp_readback.hip -- field planes from the device to host doubles, and masks from
// the host to pitched device rows.
//
// What bounds it: the host link (about 56 GB/s here) for the values, then the
// host's own pass that widens them to double. A pitched copy (hipMemcpy2D) to
// pageable memory moved a row at a time through the runtime's staging. Here a
// kernel gathers the rows of all planes, in the arithmetic type, straight into
// one of two pinned buffers while the host widens the other. Measured, float
// planes to doubles: 3 planes of 3072 x 1536 36 -> 7.5 ms, 3 planes of 24 domains
// (3.1 M nodes in all) 114 -> 3.2 ms, 7 planes of 192 x 104 x 104 536 -> 7.4 ms.
// A mask goes the other way: the host copies a share of it into one pinned buffer
// while a kernel spreads the other over the rows. The pitched copy cost 9 us per
// row: 1024 x 512 4.75 -> 0.27 ms for the whole call, and 12 admissions to a pool
// (2 masks each) 52 -> 4.9 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>

#include "lbvp_readback.h"

namespace lbvp {
namespace {

// One staging buffer's size: large enough that a launch and an event cost little
// next to its transfer, small enough to stay in the host's cache.
constexpr size_t CHUNK_BYTES = size_t(2) << 20;

struct PackArgs {
    const void* base;
    int64_t off[MAX_READ_PLANES];
    int64_t pitch;
    uint64_t first, count;     // range of the planes' values, counted row by row, plane by plane
    uint64_t per_plane;        // nx * rows
    uint32_t nx;
};

template <typename R>
__global__ void __launch_bounds__(256) k_pack(PackArgs a, R* out)
{
    const uint64_t k = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= a.count) return;
    const uint64_t e = a.first + k;
    const uint64_t q = e / a.per_plane, in = e - q * a.per_plane;
    const uint64_t row = in / a.nx;
    out[k] = static_cast<const R*>(a.base)[a.off[q] + (int64_t)row * a.pitch + (int64_t)(in - row * a.nx)];
}

// Bytes rem .. rem + count - 1 of the rows that start at dst, from in[0 .. count - 1];
// a thread reads four with one access (the link carries few small ones).
__global__ void __launch_bounds__(256) k_spread(const uint32_t* in, uint8_t* dst, int64_t pitch, uint32_t nx,
                                                uint32_t rem, uint32_t count)
{
    const uint32_t k = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (k >= count) return;
    const uint32_t v = in[k / 4];
    uint32_t row = (rem + k) / nx, col = (rem + k) - row * nx;
    const uint32_t n = min(4u, count - k);
    for (uint32_t b = 0; b < n; ++b) {
        dst[(int64_t)row * pitch + col] = (uint8_t)(v >> (8 * b));
        if (++col == nx) {
            col = 0;
            ++row;
        }
    }
}

// Two pinned buffers with an event each, of one device.
struct Staging {
    int dev = -1;
    char* p[2] = {nullptr, nullptr};
    hipEvent_t ev[2] = {nullptr, nullptr};
};

void destroy(Staging& s)
{
    for (int i = 0; i < 2; ++i) {
        if (s.ev[i]) (void)hipEventDestroy(s.ev[i]);
        if (s.p[i]) (void)hipHostFree(s.p[i]);
    }
    s = Staging{};
}

// Idle buffers: at most KEPT pairs (16 MiB), none once the last user is gone.
constexpr int KEPT = 4;
std::mutex g_mu;
Staging g_idle[KEPT];
int g_n_idle = 0;
int64_t g_users = 0;

// Buffers for work on s: its events have to be of the stream's device, which need
// not be the calling thread's current one (it stays as it was).
hipError_t acquire(hipStream_t s, Staging* out)
{
    int current = 0;
    hipError_t e = hipGetDevice(&current);
    int dev = current;   // the null stream's
    if (e == hipSuccess && s) e = hipStreamGetDevice(s, &dev);
    if (e != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        for (int i = 0; i < g_n_idle; ++i)
            if (g_idle[i].dev == dev) {
                *out = g_idle[i];
                g_idle[i] = g_idle[--g_n_idle];
                return hipSuccess;
            }
    }
    Staging st;
    st.dev = dev;
    if (dev != current) e = hipSetDevice(dev);
    for (int i = 0; i < 2 && e == hipSuccess; ++i) {
        void* m = nullptr;
        e = hipHostMalloc(&m, CHUNK_BYTES, hipHostMallocDefault);
        st.p[i] = static_cast<char*>(m);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&st.ev[i], hipEventDisableTiming);
    }
    if (dev != current) (void)hipSetDevice(current);
    if (e != hipSuccess) {
        destroy(st);
        return e;
    }
    *out = st;
    return hipSuccess;
}

// Gives a pair back; nothing enqueued may still write it.
void put_back(Staging& s)
{
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (g_users > 0 && g_n_idle < KEPT) {
            g_idle[g_n_idle++] = s;
            return;
        }
    }
    destroy(s);
}

template <typename R>
void widen(double* dst, const R* src, size_t n)
{
    for (size_t k = 0; k < n; ++k) dst[k] = (double)src[k];
}

template <typename R>
hipError_t read_typed(hipStream_t s, PackArgs a, int n, double* const* dst, Staging& st)
{
    const uint64_t total = a.per_plane * (uint64_t)n, step = CHUNK_BYTES / sizeof(R);
    auto launch = [&](uint64_t first, int slot) {
        a.first = first;
        a.count = std::min(step, total - first);
        hipLaunchKernelGGL(k_pack<R>, dim3((unsigned)((a.count + 255) / 256)), dim3(256), 0, s, a,
                           reinterpret_cast<R*>(st.p[slot]));
        const hipError_t e = hipGetLastError();
        return e != hipSuccess ? e : hipEventRecord(st.ev[slot], s);
    };
    hipError_t e = launch(0, 0);
    for (uint64_t at = 0, k = 0; at < total && e == hipSuccess; at += step, ++k) {
        const int slot = (int)(k & 1);
        if (at + step < total) e = launch(at + step, slot ^ 1);   // the other buffer fills meanwhile
        if (e == hipSuccess) e = hipEventSynchronize(st.ev[slot]);
        if (e != hipSuccess) break;
        const R* src = reinterpret_cast<const R*>(st.p[slot]);
        const uint64_t end = std::min(at + step, total);
        for (uint64_t x = at; x < end;) {   // the chunk's share of each plane
            const uint64_t q = x / a.per_plane, in = x - q * a.per_plane;
            const uint64_t len = std::min(end - x, a.per_plane - in);
            widen(dst[q] + in, src + (x - at), (size_t)len);
            x += len;
        }
    }
    return e;
}

// Where no staging buffers can be had, the pitched copies of the runtime: to
// pageable memory, a share of a plane's rows at a time.
template <typename R>
hipError_t read_pageable(hipStream_t s, const PackArgs& a, int n, double* const* dst)
{
    const size_t row = (size_t)a.nx * sizeof(R);
    const uint64_t rows = a.per_plane / a.nx, share = std::min<uint64_t>(rows, std::max<uint64_t>(1, CHUNK_BYTES / row));
    const std::unique_ptr<R[]> tmp(new (std::nothrow) R[share * a.nx]);
    if (!tmp) return hipErrorOutOfMemory;
    for (int q = 0; q < n; ++q)
        for (uint64_t r = 0; r < rows; r += share) {
            const uint64_t k = std::min(share, rows - r);
            const R* from = static_cast<const R*>(a.base) + a.off[q] + (int64_t)r * a.pitch;
            hipError_t e = hipMemcpy2DAsync(tmp.get(), row, from, (size_t)a.pitch * sizeof(R), row, (size_t)k,
                                            hipMemcpyDeviceToHost, s);
            const hipError_t w = hipStreamSynchronize(s);
            if (e == hipSuccess) e = w;
            if (e != hipSuccess) return e;
            widen(dst[q] + r * a.nx, tmp.get(), (size_t)(k * a.nx));
        }
    return hipSuccess;
}

}  // namespace

hipError_t read_planes(hipStream_t s, bool is_f64, const void* base, const int64_t* off, int n, int64_t pitch,
                       int32_t nx, int64_t rows, double* const* dst)
{
    if (n < 0 || n > MAX_READ_PLANES || nx < 1 || rows < 0) return hipErrorInvalidValue;
    if (n == 0 || rows == 0) return hipSuccess;
    PackArgs a{};
    a.base = base;
    for (int q = 0; q < n; ++q) a.off[q] = off[q];
    a.pitch = pitch;
    a.nx = (uint32_t)nx;
    a.per_plane = (uint64_t)nx * (uint64_t)rows;
    Staging st;
    hipError_t e = acquire(s, &st);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return is_f64 ? read_pageable<double>(s, a, n, dst) : read_pageable<float>(s, a, n, dst);
    }
    e = is_f64 ? read_typed<double>(s, a, n, dst, st) : read_typed<float>(s, a, n, dst, st);
    if (e != hipSuccess) (void)hipStreamSynchronize(s);   // nothing may still write the buffers
    put_back(st);
    return e;
}

hipError_t write_mask(hipStream_t s, uint8_t* dst, int64_t pitch, int32_t nx, int64_t rows, const uint8_t* src)
{
    if (nx < 1 || rows < 0) return hipErrorInvalidValue;
    if (rows == 0) return hipSuccess;
    Staging st;
    hipError_t e = acquire(s, &st);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        e = hipMemcpy2DAsync(dst, (size_t)pitch, src, (size_t)nx, (size_t)nx, (size_t)rows, hipMemcpyHostToDevice, s);
        const hipError_t w = hipStreamSynchronize(s);
        return e != hipSuccess ? e : w;
    }
    const uint64_t total = (uint64_t)nx * (uint64_t)rows;
    bool used[2] = {false, false};
    for (uint64_t at = 0, k = 0; at < total && e == hipSuccess; at += CHUNK_BYTES, ++k) {
        const int slot = (int)(k & 1);
        if (used[slot]) e = hipEventSynchronize(st.ev[slot]);
        if (e != hipSuccess) break;
        const uint32_t count = (uint32_t)std::min<uint64_t>(CHUNK_BYTES, total - at);
        std::memcpy(st.p[slot], src + at, count);
        const uint64_t row = at / (uint64_t)nx;
        hipLaunchKernelGGL(k_spread, dim3((count + 1023) / 1024), dim3(256), 0, s,
                           reinterpret_cast<const uint32_t*>(st.p[slot]), dst + (int64_t)row * pitch, pitch,
                           (uint32_t)nx, (uint32_t)(at - row * (uint64_t)nx), count);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipEventRecord(st.ev[slot], s);
        used[slot] = true;
    }
    const hipError_t w = hipStreamSynchronize(s);   // nothing may still read the buffers
    put_back(st);
    return e != hipSuccess ? e : w;
}

void readback_retain()
{
    std::lock_guard<std::mutex> lock(g_mu);
    ++g_users;
}

void readback_release()
{
    Staging gone[KEPT];
    int n = 0;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (--g_users > 0) return;
        for (n = 0; n < g_n_idle; ++n) gone[n] = g_idle[n];
        g_n_idle = 0;
    }
    for (int i = 0; i < n; ++i) destroy(gone[i]);
}

}  // namespace lbvp
