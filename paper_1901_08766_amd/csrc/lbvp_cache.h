// lbvp_cache.h -- which stores of a step are non-temporal (D2Q9 and D3Q19).
#pragma once

#include <stdint.h>

namespace lbvp {

// How many of an XCD's tiles_per_xcd tiles a launch over `bytes` of lattices (both
// of every domain) stores plain; the rest it stores non-temporal. The next step
// reads a plain result from the 256 MB last-level cache if that still holds it:
// all of them if the lattices fit. Beyond that the share that survives what the
// rest streams through shrinks to nothing at twice the cache (in between, two
// cache sizes less `bytes`: the best share of those measured lies within 32 MB of
// it). us per step with everything non-temporal, everything plain, and this share:
//   FP64 771 x 389 (43 MB)           11.7    9.1    9.1
//   FP32 2048 x 1024 moving (151 MB) 30.8   26.3   26.4
//   FP16 3840 x 1920 (265 MB)        47.9   42.4   42.3
//   FP32 192 x 104 x 104 (316 MB)    56.2   56.6   52.2
//   FP16 4096 x 2304 (340 MB)        58.7   61.0   54.8
//   FP16 5120 x 2560 (472 MB)        80.7   83.8   78.9
//   FP16 8192 x 4096 (1.2 GB)       200.0  200.1  200.1 (FP32 step 3% slower if plain)
inline int32_t keep_tiles(uint64_t bytes, int32_t tiles_per_xcd)
{
    constexpr uint64_t CACHE = uint64_t(1) << 28;
    if (bytes <= CACHE) return tiles_per_xcd;
    if (bytes >= 2 * CACHE) return 0;
    return (int32_t)((double)(2 * CACHE - bytes) / (double)bytes * tiles_per_xcd);
}

}  // namespace lbvp
