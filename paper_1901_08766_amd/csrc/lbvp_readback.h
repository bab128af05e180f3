// lbvp_readback.h -- field planes from the device to host doubles and masks from
// the host to pitched device rows, shared by the D2Q9 and D3Q19 calls.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace lbvp {

constexpr int MAX_READ_PLANES = 7;

// Reads `rows` rows of nx values from each of n planes of a pitched device array
// (arithmetic type: double if is_f64, else float; plane q starts at element
// off[q]) into dst[q], rows back to back. Enqueues on s and waits for it.
hipError_t read_planes(hipStream_t s, bool is_f64, const void* base, const int64_t* off, int n, int64_t pitch,
                       int32_t nx, int64_t rows, double* const* dst);

// Writes `rows` rows of nx bytes, back to back at src, to device rows of `pitch`
// bytes (the rest of a row is left as it is). Enqueues on s; src has been read
// when it returns.
hipError_t write_mask(hipStream_t s, uint8_t* dst, int64_t pitch, int32_t nx, int64_t rows, const uint8_t* src);

// The pinned staging buffers that both use are kept between calls while
// any context or pool lives: each counts itself in and out.
void readback_retain();
void readback_release();
struct ReadbackUser {
    ReadbackUser() { readback_retain(); }
    ~ReadbackUser() { readback_release(); }
    ReadbackUser(const ReadbackUser&) = delete;
    ReadbackUser& operator=(const ReadbackUser&) = delete;
};

}  // namespace lbvp
