// lbvp_kernels.hip -- the kernels next to the D2Q9 step: record sums on their own,
// initialization and conversions between the stored populations and host values,
// the AA layout's ghost columns, halo columns of slab cuts, and the plain copy;
// and the dispatch of step launches to the storage types' translation units.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lbvp_device.h"
#include "lbvp_internal.h"
#include "lbvp_node.h"

namespace lbvp {
namespace {

// The last records of an lbvp_step call, summed on their own.
__global__ void __launch_bounds__(FIN_THREADS) k_finalize(FinalizeArgs a, int32_t buf, int32_t n)
{
    __shared__ double lds[2 * FIN_LANES];
    finalize_record(a, buf, n, (int)blockIdx.x, FIN_COUNTERS, lds);
}

// The same for every domain of a batch.
__global__ void __launch_bounds__(FIN_THREADS) k_finalize_batch(const FinalizeArgs* fins, int32_t share, int32_t buf)
{
    __shared__ double lds[2 * FIN_LANES];
    const int d = (int)blockIdx.x / share;
    finalize_record(fins[d], buf, 1, (int)blockIdx.x - d * share, share, lds);
}

// Moving bodies: after a run of n steps, the pose table row of the next step.
__global__ void k_pose_advance(int64_t* base, int64_t n) { *base += n; }

template <typename R>
__global__ void __launch_bounds__(256) k_pose_advance_batch(const StepArgs<R>* args, int32_t n_domains, int64_t n)
{
    const int d = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (d < n_domains && args[d].n_moving > 0) *const_cast<int64_t*>(args[d].pose_base) += n;
}

// ------------------------------------------------------------ conversions --
__constant__ double W_ALL[9] = {4.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0,
                                1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0};
__constant__ int EX_ALL[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__constant__ int EY_ALL[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
__constant__ int OPP_ALL[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};

// Algorithm step (1): populations at equilibrium (eq. feq) for staged rows, in
// FP64, stored as normalized deviations; the fields of step 0 are (rho, u, 0, 0).
// In the AA layout the post-collision population q of a node lives in its slot
// opp(q) after an even number of steps (a.swap).
template <typename S>
__global__ void __launch_bounds__(256) k_init(S* lat, typename Arith<S>::R* fields, ConvArgs a)
{
    using R = typename Arith<S>::R;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)a.rows * a.nx) return;
    const int jl = (int)(k / a.nx), i = (int)(k - (int64_t)jl * a.nx);
    const double rho = a.rho ? a.rho[k] : a.rho0;
    const double ux = a.ux ? a.ux[k] : 0.0;
    const double uy = a.uy ? a.uy[k] : 0.0;
    const double uu = ux * ux + uy * uy;
    const int64_t o = (int64_t)(a.row0 + jl) * a.pitch + i;
    const int64_t lo = (int64_t)(a.row0 + jl) * a.lstride + i;
    for (int q = 0; q < 9; ++q) {
        const double eu = EX_ALL[q] * ux + EY_ALL[q] * uy;
        const double h = (rho - a.rho0) + rho * (3.0 * eu + 4.5 * eu * eu - 1.5 * uu);
        lat[(a.swap ? OPP_ALL[q] : q) * a.plane + lo] = enc<S>((R)h);
    }
    if (fields) {
        fields[o] = (R)rho;
        fields[a.plane_f + o] = (R)ux;
        fields[2 * a.plane_f + o] = (R)uy;
        fields[3 * a.plane_f + o] = R(0);
        fields[4 * a.plane_f + o] = R(0);
    }
}

template <typename S>
__global__ void __launch_bounds__(256) k_decode(const S* lat, ConvArgs a)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)a.rows * a.nx;
    if (k >= n) return;
    const int jl = (int)(k / a.nx), i = (int)(k - (int64_t)jl * a.nx);
    const int64_t lo = (int64_t)(a.row0 + jl) * a.lstride + i;
    for (int q = 0; q < 9; ++q)
        a.pops[q * n + k] = W_ALL[q] * ((double)dec(lat[(a.swap ? OPP_ALL[q] : q) * a.plane + lo]) + a.rho0);
}

template <typename S>
__global__ void __launch_bounds__(256) k_encode(S* lat, ConvArgs a)
{
    using R = typename Arith<S>::R;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)a.rows * a.nx;
    if (k >= n) return;
    const int jl = (int)(k / a.nx), i = (int)(k - (int64_t)jl * a.nx);
    const int64_t lo = (int64_t)(a.row0 + jl) * a.lstride + i;
    for (int q = 0; q < 9; ++q)
        lat[(a.swap ? OPP_ALL[q] : q) * a.plane + lo] = enc<S>((R)(a.pops[q * n + k] / W_ALL[q] - a.rho0));
}

__global__ void k_set_i64(int64_t* p, int64_t v) { p[threadIdx.x] = v; }

// A plain device copy: one 16-byte non-temporal load and store per thread in
// 64-thread blocks, the fastest of the copy forms measured (6.6-6.7 TB/s against
// 6.1 for four elements per thread in 256-thread blocks, XCD-ordered or not):
// the bandwidth the memory system gives a streaming read-and-write, against
// which the steps are measured.
__global__ void __launch_bounds__(64) k_copy16(const u32x4_t* __restrict__ src, u32x4_t* __restrict__ dst, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (i < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// AA layout after an even number of steps: copy the outflow sides' outgoing
// post-collision populations into the ghost columns the next push step reads.
template <typename S>
__global__ void __launch_bounds__(256) k_aa_ghosts(const S* lat, GhostArgs a)
{
    const int y = blockIdx.x * blockDim.x + threadIdx.x;
    if (y >= a.ny) return;
    const int64_t row = (int64_t)y * a.lstride;
    const int exp_q[3] = {1, 5, 8}, exm_q[3] = {3, 6, 7};
    for (int m = 0; m < 3; ++m) {
        if (a.west_outflow)
            static_cast<S*>(a.ghost_w)[m * (int64_t)a.ny + y] = lat[OPP_ALL[exp_q[m]] * a.plane + row];
        if (a.east_outflow)
            static_cast<S*>(a.ghost_e)[m * (int64_t)a.ny + y] = lat[OPP_ALL[exm_q[m]] * a.plane + row + a.nx - 1];
    }
}

// The halo columns of every cut of a slab decomposition (one thread per row and
// direction of each link): plain copies of the storage values, so that a
// decomposed domain steps bitwise like the whole one.
template <typename S>
__global__ void __launch_bounds__(256) k_halo(HaloArgs h)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per_link = 3 * (int64_t)h.ny;
    if (k >= per_link * h.n_links) return;
    const int l = (int)(k / per_link);
    const int r = (int)(k - (int64_t)l * per_link);
    const int m = r / h.ny, j = r - m * h.ny;
    const HaloLink& L = h.link[l];
    const int q_in = m == 0 ? 1 : (m == 1 ? 5 : 8);    // e_x = +1 (1, 5, 8): leave west through its east side
    const int q_out = m == 0 ? 3 : (m == 1 ? 6 : 7);   // e_x = -1 (3, 6, 7): leave east through its west side
    const S* wl = static_cast<const S*>(L.w_lat);
    const S* el = static_cast<const S*>(L.e_lat);
    // east slab's west halo: its last padding column; west slab's east halo: column nx
    static_cast<S*>(L.e_lat_w)[j * L.e_lstride + q_in * L.e_plane + (L.e_pitch - 1)] =
        wl[j * L.w_lstride + q_in * L.w_plane + (L.w_nx - 1)];
    static_cast<S*>(L.w_lat_w)[j * L.w_lstride + q_out * L.w_plane + L.w_nx] = el[j * L.e_lstride + q_out * L.e_plane];
}

// The same for the cuts of a batch, before one of its steps: each member's
// current lattice is read from its step arguments (so a captured graph replays
// correctly whatever the members' lattice parity when it is launched).
template <typename S>
__global__ void __launch_bounds__(256) k_halo_batch(BatchHalo h)
{
    using R = typename Arith<S>::R;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per_link = 3 * (int64_t)h.ny;
    if (k >= per_link * h.n_links) return;
    const int l = (int)(k / per_link);
    const int r = (int)(k - (int64_t)l * per_link);
    const int m = r / h.ny, j = r - m * h.ny;
    const StepArgs<R>* args = static_cast<const StepArgs<R>*>(h.args);
    const StepArgs<R>& aw = args[h.w[l]];
    const StepArgs<R>& ae = args[h.e[l]];
    S* wl = static_cast<S*>((aw.cur ^ h.flip) ? aw.lat1 : aw.lat0);
    S* el = static_cast<S*>((ae.cur ^ h.flip) ? ae.lat1 : ae.lat0);
    const int q_in = m == 0 ? 1 : (m == 1 ? 5 : 8);
    const int q_out = m == 0 ? 3 : (m == 1 ? 6 : 7);
    el[j * ae.lstride + q_in * ae.plane + (ae.pitch - 1)] = wl[j * aw.lstride + q_in * aw.plane + (aw.nx - 1)];
    wl[j * aw.lstride + q_out * aw.plane + aw.nx] = el[j * ae.lstride + q_out * ae.plane];
}

unsigned conv_blocks(const ConvArgs& a) { return (unsigned)(((int64_t)a.rows * a.nx + 255) / 256); }

}  // namespace

int vector_width(int32_t storage)
{
    switch (storage) {
    case ST_F64: return 2;
    case ST_F32: return 4;
    default: return 8;
    }
}

hipError_t launch_step(int32_t storage, int32_t mode, bool record, bool fields, const void* src, void* dst,
                       const void* step_args, hipStream_t s)
{
    switch (storage) {
    case ST_F64: return StepLaunch<double>::one(false, mode, record, fields, src, dst, step_args, s);
    case ST_F32: return StepLaunch<float>::one(false, mode, record, fields, src, dst, step_args, s);
    case ST_F16: return StepLaunch<_Float16>::one(false, mode, record, fields, src, dst, step_args, s);
    case ST_BF16: return StepLaunch<__bf16>::one(false, mode, record, fields, src, dst, step_args, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step_moving(int32_t storage, int32_t mode, bool record, bool fields, const void* src, void* dst,
                              const void* step_args, hipStream_t s)
{
    switch (storage) {
    case ST_F64: return StepLaunch<double>::one(true, mode, record, fields, src, dst, step_args, s);
    case ST_F32: return StepLaunch<float>::one(true, mode, record, fields, src, dst, step_args, s);
    case ST_F16: return StepLaunch<_Float16>::one(true, mode, record, fields, src, dst, step_args, s);
    case ST_BF16: return StepLaunch<__bf16>::one(true, mode, record, fields, src, dst, step_args, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step_batch(int32_t storage, int32_t vec, int32_t block, int32_t mode, bool record, bool fields,
                             bool moving, const BatchLaunch& b, hipStream_t s)
{
    switch (storage) {
    case ST_F64: return StepLaunch<double>::batch(moving, vec, block, mode, record, fields, b, s);
    case ST_F32: return StepLaunch<float>::batch(moving, vec, block, mode, record, fields, b, s);
    case ST_F16: return StepLaunch<_Float16>::batch(moving, vec, block, mode, record, fields, b, s);
    case ST_BF16: return StepLaunch<__bf16>::batch(moving, vec, block, mode, record, fields, b, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_march(int32_t storage, const void* src, void* dst, const void* step_args, const MarchArgs& m,
                        hipStream_t s)
{
    switch (storage) {
    case ST_F64: return MarchLaunch<double>::one(src, dst, step_args, m, s);
    case ST_F32: return MarchLaunch<float>::one(src, dst, step_args, m, s);
    default: return hipErrorInvalidValue;   // 2-byte storage runs single steps
    }
}

hipError_t launch_pose_advance(int64_t* base, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_pose_advance, dim3(1), dim3(1), 0, s, base, n);
    return hipGetLastError();
}

hipError_t launch_pose_advance_batch(int32_t storage, const void* args, int32_t n_domains, int64_t n, hipStream_t s)
{
    const dim3 g((unsigned)((n_domains + 255) / 256)), b(256);
    if (storage == ST_F64)
        hipLaunchKernelGGL(k_pose_advance_batch<double>, g, b, 0, s, static_cast<const StepArgs<double>*>(args),
                           n_domains, n);
    else
        hipLaunchKernelGGL(k_pose_advance_batch<float>, g, b, 0, s, static_cast<const StepArgs<float>*>(args),
                           n_domains, n);
    return hipGetLastError();
}

// Few domains: their launches are short, so a record's sums run side by side
// (as for a single domain); many domains already spread theirs over the chip.
int32_t batch_fin_share(int32_t n) { return n <= 16 ? 4 : n <= 64 ? 2 : 1; }

hipError_t launch_finalize_batch(const FinalizeArgs* fin_dev, int32_t n, int32_t buf, hipStream_t s)
{
    const int32_t share = batch_fin_share(n);
    hipLaunchKernelGGL(k_finalize_batch, dim3((unsigned)(n * share)), dim3(FIN_THREADS), 0, s, fin_dev, share, buf);
    return hipGetLastError();
}

hipError_t launch_aa_ghosts(int32_t storage, const void* lat, const GhostArgs& a, hipStream_t s)
{
    const dim3 g((unsigned)((a.ny + 255) / 256)), b(256);
    switch (storage) {
    case ST_F64: hipLaunchKernelGGL(k_aa_ghosts<double>, g, b, 0, s, (const double*)lat, a); break;
    case ST_F32: hipLaunchKernelGGL(k_aa_ghosts<float>, g, b, 0, s, (const float*)lat, a); break;
    case ST_F16: hipLaunchKernelGGL(k_aa_ghosts<_Float16>, g, b, 0, s, (const _Float16*)lat, a); break;
    case ST_BF16: hipLaunchKernelGGL(k_aa_ghosts<__bf16>, g, b, 0, s, (const __bf16*)lat, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_finalize(const FinalizeArgs& a, int32_t buf, int32_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize, dim3(FIN_COUNTERS), dim3(FIN_THREADS), 0, s, a, buf, n);
    return hipGetLastError();
}

hipError_t launch_init(int32_t storage, void* lat, void* fields, const ConvArgs& a, hipStream_t s)
{
    const dim3 g(conv_blocks(a)), b(256);
    switch (storage) {
    case ST_F64: hipLaunchKernelGGL(k_init<double>, g, b, 0, s, (double*)lat, (double*)fields, a); break;
    case ST_F32: hipLaunchKernelGGL(k_init<float>, g, b, 0, s, (float*)lat, (float*)fields, a); break;
    case ST_F16: hipLaunchKernelGGL(k_init<_Float16>, g, b, 0, s, (_Float16*)lat, (float*)fields, a); break;
    case ST_BF16: hipLaunchKernelGGL(k_init<__bf16>, g, b, 0, s, (__bf16*)lat, (float*)fields, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_decode(int32_t storage, const void* lat, const ConvArgs& a, hipStream_t s)
{
    const dim3 g(conv_blocks(a)), b(256);
    switch (storage) {
    case ST_F64: hipLaunchKernelGGL(k_decode<double>, g, b, 0, s, (const double*)lat, a); break;
    case ST_F32: hipLaunchKernelGGL(k_decode<float>, g, b, 0, s, (const float*)lat, a); break;
    case ST_F16: hipLaunchKernelGGL(k_decode<_Float16>, g, b, 0, s, (const _Float16*)lat, a); break;
    case ST_BF16: hipLaunchKernelGGL(k_decode<__bf16>, g, b, 0, s, (const __bf16*)lat, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_encode(int32_t storage, void* lat, const ConvArgs& a, hipStream_t s)
{
    const dim3 g(conv_blocks(a)), b(256);
    switch (storage) {
    case ST_F64: hipLaunchKernelGGL(k_encode<double>, g, b, 0, s, (double*)lat, a); break;
    case ST_F32: hipLaunchKernelGGL(k_encode<float>, g, b, 0, s, (float*)lat, a); break;
    case ST_F16: hipLaunchKernelGGL(k_encode<_Float16>, g, b, 0, s, (_Float16*)lat, a); break;
    case ST_BF16: hipLaunchKernelGGL(k_encode<__bf16>, g, b, 0, s, (__bf16*)lat, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_copy16(const void* src, void* dst, int64_t n16, hipStream_t s)
{
    const int64_t blocks = (n16 + 63) / 64;
    if (blocks > (int64_t(1) << 31) - 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(64), 0, s, static_cast<const u32x4_t*>(src),
                       static_cast<u32x4_t*>(dst), n16);
    return hipGetLastError();
}

hipError_t launch_halo(int32_t storage, const HaloArgs& h, hipStream_t s)
{
    const int64_t n = 3 * (int64_t)h.ny * h.n_links;
    const dim3 g((unsigned)((n + 255) / 256)), b(256);
    switch (storage) {
    case ST_F64: hipLaunchKernelGGL(k_halo<double>, g, b, 0, s, h); break;
    case ST_F32: hipLaunchKernelGGL(k_halo<float>, g, b, 0, s, h); break;
    case ST_F16: hipLaunchKernelGGL(k_halo<_Float16>, g, b, 0, s, h); break;
    case ST_BF16: hipLaunchKernelGGL(k_halo<__bf16>, g, b, 0, s, h); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_halo_batch(int32_t storage, const BatchHalo& h, hipStream_t s)
{
    const int64_t n = 3 * (int64_t)h.ny * h.n_links;
    const dim3 g((unsigned)((n + 255) / 256)), b(256);
    switch (storage) {
    case ST_F64: hipLaunchKernelGGL(k_halo_batch<double>, g, b, 0, s, h); break;
    case ST_F32: hipLaunchKernelGGL(k_halo_batch<float>, g, b, 0, s, h); break;
    case ST_F16: hipLaunchKernelGGL(k_halo_batch<_Float16>, g, b, 0, s, h); break;
    case ST_BF16: hipLaunchKernelGGL(k_halo_batch<__bf16>, g, b, 0, s, h); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_set_i64(int64_t* p, int32_t n, int64_t v, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_i64, dim3(1), dim3((unsigned)n), 0, s, p, v);
    return hipGetLastError();
}

}  // namespace lbvp
