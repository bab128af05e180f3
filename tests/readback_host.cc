// readback_host.cc -- the host side of csrc/lbvp_readback.hip on the stand-in runtime.
// usage: readback_host CHECK; exits with 0 if it holds.
#include "fake_hip.h"
#include "lbvp_readback.h"

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
