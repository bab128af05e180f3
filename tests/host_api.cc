// host_api.cc -- the host side of the D2Q9 calls (contexts, batches, the pool) on the
// stand-in runtime, with launches that do nothing.
// usage: host_api CHECK; exits with 0 if it holds.
#include "fake_hip.h"
#include "lbvp.h"
#include "lbvp_internal.h"

#include <array>

namespace lbvp {
int vector_width(int32_t storage) { return storage == ST_F64 ? 2 : storage == ST_F32 ? 4 : 8; }
int32_t batch_fin_share(int32_t) { return 1; }
hipError_t launch_march(int32_t, const void*, void*, const void*, const MarchArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_step(int32_t, int32_t, bool, bool, const void*, void*, const void*, hipStream_t) { return hipSuccess; }
hipError_t launch_step_moving(int32_t, int32_t, bool, bool, const void*, void*, const void*, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_aa_ghosts(int32_t, const void*, const GhostArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_step_batch(int32_t, int32_t, int32_t, int32_t, bool, bool, bool, const BatchLaunch&, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_pose_advance(int64_t*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_pose_advance_batch(int32_t, const void*, int32_t, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_finalize_batch(const FinalizeArgs*, int32_t, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_finalize(const FinalizeArgs&, int32_t, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_init(int32_t, void*, void*, const ConvArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_decode(int32_t, const void*, const ConvArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_encode(int32_t, void*, const ConvArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_set_i64(int64_t*, int32_t, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_copy16(const void*, void*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_halo(int32_t, const HaloArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_halo_batch(int32_t, const BatchHalo&, hipStream_t) { return hipSuccess; }
}  // namespace lbvp

static lbvp_params params(int32_t nx, int32_t ny, int32_t storage)
{
    lbvp_params p{};
    p.nx = nx;
    p.ny = ny;
    p.tau_plus = 0.8;
    p.magic_lambda = 0.25;
    p.eta = 1e-4;
    p.rho0 = 1.0;
    p.storage = storage;
    p.force_every = 1;
    p.force_capacity = 64;
    p.max_bodies = 4;
    return p;
}

// A pool that serves one request at a time keeps its staging buffers in between, and
// gives them back when it goes.
static int pool_staging()
{
    ihipStream_t s{0};
    lbvp_pool_config cfg{};
    cfg.cap_bytes = size_t(1) << 30;
    cfg.chunk_bytes = size_t(64) << 20;
    cfg.max_slots = 2;
    cfg.storage = LBVP_F32;
    lbvp_pool* p = nullptr;
    CHECK(lbvp_pool_create(&cfg, &s, &p) == LBVP_OK);
    const lbvp_params prm = params(64, 32, LBVP_F32);
    const std::vector<uint8_t> mask(64 * 32, 0);
    for (int k = 0; k < 6; ++k) {
        int32_t slot = -1;
        const lbvp_status st = lbvp_pool_admit(p, &prm, mask.data(), 0, nullptr, nullptr, nullptr, nullptr, 4, &slot);
        if (st != LBVP_OK) std::printf("admit: %s\n", lbvp_pool_last_error(p));
        CHECK(st == LBVP_OK);
        CHECK(lbvp_pool_release(p, slot) == LBVP_OK);
        CHECK(fake::host_allocs == 2);
    }
    CHECK(lbvp_pool_destroy(p) == LBVP_OK);
    CHECK(fake::host_frees == fake::host_allocs);
    return 0;
}

// Members whose tables fill the 4 MiB array of lbvp_batch_step_static: as many as ever
// fit (648 bytes of arguments a member in FP64, 536 in FP32, a tile and its start), and
// no more.
static int static_capacity()
{
    ihipStream_t s{0};
    for (const auto& [storage, fit, refused] : {std::array<int, 3>{LBVP_F64, 6390, 6400}, {LBVP_F32, 7700, 7720}}) {
        const lbvp_params p = params(3, 3, storage);
        const size_t n = lbvp_footprint_bytes(&p);
        void* mem = nullptr;
        CHECK(hipMalloc(&mem, n) == hipSuccess);
        std::vector<lbvp_ctx*> c((size_t)refused, nullptr);
        for (lbvp_ctx*& x : c) CHECK(lbvp_create(&p, &s, mem, n, &x) == LBVP_OK);   // nothing runs: one memory for all
        CHECK(lbvp_batch_step_static(c.data(), fit, 1, 0) == LBVP_OK);
        CHECK(lbvp_batch_step_static(c.data(), refused, 1, 0) == LBVP_E_ARG);
        for (lbvp_ctx* x : c) CHECK(lbvp_destroy(x) == LBVP_OK);
        hipFree(mem);
    }
    return 0;
}

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "pool_staging")) return pool_staging();
    if (!std::strcmp(what, "static_capacity")) return static_capacity();
    std::printf("unknown check %s\n", what);
    return 2;
}
