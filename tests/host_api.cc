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
// fit (648 bytes of arguments a member in FP64 and 536 in FP32 at most, a tile and its
// start), and
// no more.
static int static_capacity()
{
    ihipStream_t s{0};
    for (const auto& [storage, fit, refused] : {std::array<int, 3>{LBVP_F64, 6390, 6480}, {LBVP_F32, 7700, 7840}}) {
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

// A ragged 2-byte grid whose default shape has smaller blocks than the 256 threads of
// other grids is still taken wherever a context of 256 would be: next to their defaults
// in lbvp_batch_step_static, with undrained records where its shape becomes (4, 256), and
// with as many (tile, body) pairs.
static int default_shape()
{
    ihipStream_t s{0};
    lbvp_params a = params(2305, 1153, LBVP_F16_DEV), b = params(2048, 1200, LBVP_F16_DEV);
    a.max_bodies = 20;
    auto make = [&](const lbvp_params& p) {
        lbvp_ctx* c = nullptr;
        return lbvp_create(&p, &s, nullptr, 0, &c) == LBVP_OK ? c : nullptr;
    };
    auto is = [](const lbvp_ctx* c, int32_t v, int32_t k) {
        int32_t vec = 0, block = 0;
        return lbvp_get_launch(c, &vec, &block) == LBVP_OK && vec == v && block == k;
    };
    lbvp_ctx *m[2] = {make(a), make(b)}, *same[2] = {make(a), make(a)}, *later[2] = {m[1], make(a)};
    CHECK(m[0] && m[1] && same[0] && same[1] && later[1]);
    CHECK(is(m[0], 4, 128) && is(m[1], 4, 256));
    CHECK(lbvp_step(m[0], 3, 0) == LBVP_OK);
    CHECK(lbvp_batch_step_static(m, 2, 1, 0) == LBVP_OK);
    CHECK(is(m[0], 4, 256) && is(m[1], 4, 256));
    CHECK(lbvp_step(m[0], 1, 0) == LBVP_OK);
    CHECK(lbvp_batch_step_static(later, 2, 1, 0) == LBVP_OK);
    // shapes that agree stay; a set one is not changed, nor is anything by a refused call
    CHECK(lbvp_batch_step_static(same, 2, 1, 0) == LBVP_OK && is(same[0], 4, 128) && is(same[1], 4, 128));
    lbvp_ctx *fixed = make(a), *open = make(a), *bad[3] = {m[1], fixed, open};
    CHECK(fixed && open && lbvp_set_launch(fixed, 4, 128) == LBVP_OK);
    CHECK(lbvp_batch_step_static(bad, 3, 1, 0) == LBVP_E_ARG);
    CHECK(is(fixed, 4, 128) && is(open, 4, 128));
    // undrained records
    lbvp_ctx *c = make(a), *d = make(a);
    CHECK(c && lbvp_step(c, 3, 0) == LBVP_OK);
    CHECK(lbvp_set_launch(c, 4, 64) == LBVP_E_STATE);
    CHECK(lbvp_set_launch(c, 8, 256) == LBVP_E_STATE);
    lbvp_batch* batch = nullptr;
    CHECK(lbvp_batch_create(&c, 1, 4, 256, &batch) == LBVP_OK);
    CHECK(lbvp_batch_step(batch, 2, 0) == LBVP_OK);
    CHECK(lbvp_batch_destroy(batch) == LBVP_OK);
    CHECK(d && lbvp_step(d, 3, 0) == LBVP_OK);
    CHECK(lbvp_set_launch(d, 4, 256) == LBVP_OK && is(d, 4, 256));
    CHECK(lbvp_set_launch(d, 4, 128) == LBVP_E_STATE);
    // 20 bodies in every tile: room for that many pairs in tiles of (4, 256) only
    std::vector<uint8_t> mask((size_t)a.nx * a.ny);
    for (size_t k = 0; k < mask.size(); ++k) mask[k] = (uint8_t)(k % a.nx % 20 + 1);
    const std::vector<lbvp_body> bodies(20, lbvp_body{});
    lbvp_ctx* e = make(a);
    CHECK(e && lbvp_set_mask(e, mask.data(), 20, bodies.data()) == LBVP_OK && is(e, 4, 256));
    CHECK(lbvp_step(e, 3, 0) == LBVP_OK);
    CHECK(lbvp_set_launch(fixed, 4, 64) == LBVP_OK);
    CHECK(lbvp_set_mask(fixed, mask.data(), 20, bodies.data()) == LBVP_E_NOMEM);
    for (lbvp_ctx* x : {m[0], m[1], same[0], same[1], later[1], fixed, open, c, d, e}) CHECK(lbvp_destroy(x) == LBVP_OK);
    return 0;
}

// The tuner's cached rows of a domain are not those of a slab of its size, whose cut
// keeps it from running two steps a launch, and the other way round.
static int tune_cuts()
{
    ihipStream_t s{0};
    lbvp_params whole = params(256, 128, LBVP_F32), slab = whole;
    slab.bc_west = slab.bc_east = LBVP_BC_NEIGHBOR;
    whole.bc_west = whole.bc_east = LBVP_BC_PERIODIC;
    slab.force_capacity = whole.force_capacity = 1024;
    lbvp_ctx *w = nullptr, *c = nullptr;
    CHECK(lbvp_create(&whole, &s, nullptr, 0, &w) == LBVP_OK);
    CHECK(lbvp_create(&slab, &s, nullptr, 0, &c) == LBVP_OK);
    lbvp_tune_row rows[32];
    auto measures = [&](lbvp_ctx* x) {   // whether the call made scratch contexts
        int32_t n = 0, best = 0;
        const int before = fake::dev_allocs;
        const lbvp_status st = lbvp_tune(&x, 1, 4, 0, rows, 32, &n, &best);
        if (st != LBVP_OK) std::printf("%s\n", lbvp_tune_last_error());
        return st != LBVP_OK ? -1 : fake::dev_allocs > before ? 1 : 0;
    };
    CHECK(measures(w) == 1);
    CHECK(measures(c) == 1);
    CHECK(measures(w) == 0);
    CHECK(measures(c) == 0);
    CHECK(lbvp_destroy(w) == LBVP_OK && lbvp_destroy(c) == LBVP_OK);
    return 0;
}

// Default blocks of 2-byte grids: 128 threads for 256 on ragged grids well within the
// last-level cache, 256 where they pad as little or the lattices come close to its size,
// never 64 for a grid of this many nodes.
static int default_blocks()
{
    ihipStream_t s{0};
    struct { int32_t nx, ny, block; } cases[] = {{1030, 2135, 128}, {1100, 5000, 128}, {2305, 2819, 128}, {4110, 1581, 128},
                                                 {1030, 7087, 256}, {2567, 2891, 256}, {2305, 3167, 256}, {1550, 2258, 256},
                                                 {2567, 857, 256}, {2048, 1200, 256}, {4100, 2100, 256}};
    for (int32_t storage : {LBVP_F16_DEV, LBVP_BF16_DEV})
        for (const auto& k : cases) {
            const lbvp_params p = params(k.nx, k.ny, storage);
            lbvp_ctx* c = nullptr;
            int32_t vec = 0, block = 0;
            CHECK(lbvp_create(&p, &s, nullptr, 0, &c) == LBVP_OK && lbvp_get_launch(c, &vec, &block) == LBVP_OK);
            if (vec != 4 || block != k.block) std::printf("%d x %d: (%d, %d)\n", k.nx, k.ny, vec, block);
            CHECK(vec == 4 && block == k.block);
            CHECK(lbvp_destroy(c) == LBVP_OK);
        }
    return 0;
}

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "pool_staging")) return pool_staging();
    if (!std::strcmp(what, "static_capacity")) return static_capacity();
    if (!std::strcmp(what, "default_shape")) return default_shape();
    if (!std::strcmp(what, "tune_cuts")) return tune_cuts();
    if (!std::strcmp(what, "default_blocks")) return default_blocks();
    std::printf("unknown check %s\n", what);
    return 2;
}
