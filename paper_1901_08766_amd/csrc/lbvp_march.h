// lbvp_march.h -- two D2Q9 time steps in one pass over the lattice, for FP64 and
// FP32 vector launches: instantiated by lbvp_march_f64.hip and lbvp_march_f32.hip.
//
// A single step is bound by its 18 lattice values per node, read and written
// once. Two steps fused move the same bytes for twice the updates: a workgroup
// takes a strip of the width of a tile (vec * block columns) and marches up a
// chunk of its rows. At each row it does the first step of row r (from the source
// lattice, as a single step would) and then the second step of row r - 1, whose
// streamed populations are the first step's results of rows r - 2, r - 1 and r in
// its own columns. Rows r - 2 and r - 1 wait in LDS, in the slots of the thread that
// owns the columns; x neighbours come by lane shifts. Only the columns at a
// wavefront's ends are exchanged through LDS, and the two columns next to the
// strip, whose first step the workgroup computes itself for all rows of the chunk
// before it marches. A chunk of H rows does the first step of H + 2.
//
// The first step's results are rounded to the storage type and every node's
// arithmetic is that of the single step, so the lattice after a pass is bitwise
// that of two single steps. Both steps' records use the single step's partials
// (wavefront and tile of the launch shape), in the same order, so they are too.
//
// What bounds it now is a wavefront's chain of rows (loads, 9 V values of first
// step, barrier, 9 V of second step, stores) with 3 wavefronts per SIMD to hide it:
// 142 (FP32) and 145 (FP64) registers, and 9 results of every column in LDS (25 KB
// per 128 threads). Against single steps with the same stores, us per step: FP32 3072 x
// 1536 43.0 for 54.9, at 48 % of the vector unit's rate and half of the memory's; FP64
// 2305 x 1153 50.3 for 65.0; the 8192 x 4096 five-body domain 232 for 387 and 446 for 776.
// Measured and left out (FP32 3072 x 1536 with every store non-temporal, against 46.0):
// the held rows in registers (208
// of them, 2 wavefronts: 52), loads of the next row ahead of the first step's arithmetic
// (182 registers: 49), registers cut to 4 wavefronts (54).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lbvp_device.h"
#include "lbvp_internal.h"
#include "lbvp_node.h"

namespace lbvp {
namespace {

// The source lattice's populations of V nodes of a row as the step reads them:
// FP32 vectors take the x-shifted directions one element off; FP64 vectors load
// aligned and keep the end elements apart.
template <typename S, int V>
struct RowLoad {
    static constexpr bool kShifted = sizeof(S) == 4;
    S v[9][V];
    S left[3], right[3];   // !kShifted: column i0 - 1 of EXP, i0 + V of EXM
};

// Tables that no launch changes, at a uniform index: scalar loads that no store of
// the pass can alias.
template <typename T>
__device__ __forceinline__ T table_at(const T* p, int64_t i)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using C = const __attribute__((address_space(4))) T;
    return ((C*)p)[i];
#else
    return p[i];
#endif
}

// A value that is the same in every lane, in scalar registers from here on: a
// quotient, which only the vector unit computes, would drag all arithmetic on it
// there, and the loop optimizer would turn every access at a scalar offset into a
// vector pointer of its own (18 register pairs).
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform(int64_t x)
{
    const uint32_t lo = (uint32_t)uniform((int)(uint32_t)x), hi = (uint32_t)uniform((int)(uint32_t)((uint64_t)x >> 32));
    return (int64_t)((uint64_t)hi << 32 | lo);
}

// A value the optimizer may not look through: what is computed from it stays where
// it is written, instead of being computed ahead of the loop and kept in (spilled)
// registers for the few waves that need it.
__device__ __forceinline__ int opaque(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// The kernel's StepArgs (after two pointers), to be read again where a value is
// needed once a row.
template <typename R>
struct KernelArgs {
#if defined(__HIP_DEVICE_COMPILE__)
    using T = const __attribute__((address_space(4))) StepArgs<R>;
    __device__ __forceinline__ T* get() const
    {
        T* p = (T*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + 16);
        asm volatile("" : "+s"(p));
        return p;
    }
#else
    __host__ __device__ const StepArgs<R>* get() const { return nullptr; }
#endif
};

// Direction q pulls from lattice row j - e_y: 0 for e_y = 0, 1 for +1, 2 for -1.
constexpr int ROWQ[9] = {0, 0, 1, 0, 2, 1, 1, 2, 2};

// The lattice rows a row pulls from, by ROWQ, as element offsets.
struct Rows3 {
    int64_t o[3];
};

template <typename R>
__device__ __forceinline__ Rows3 rows_of(int j, const StepArgs<R>& a)
{
    const int jm = j == 0 ? a.ny - 1 : j - 1, jp = j == a.ny - 1 ? 0 : j + 1;
    return {{(int64_t)j * a.lstride, (int64_t)jm * a.lstride, (int64_t)jp * a.lstride}};
}

// The two x sides as a strip's loads see them: the column that stands in for the
// one outside the domain, or -1 for an inflow, whose populations in the storage
// type (EXP of a west side, EXM of an east one) the workgroup keeps in LDS.
struct Sides {
    int west_col, east_col;
};

// Population value at row[off + col], or inflow[m] (LDS) for col = -1; both are
// read, so that each keeps its own kind of load.
template <typename S>
__device__ __forceinline__ S side_value(const S* row, int64_t off, int col, const S (&inflow)[3], int m)
{
    const S in = inflow[m];
    const S x = row[off + max(col, 0)];
    return col < 0 ? in : x;
}

// The value of a storage element as the bits of a 32-bit lane register and back,
// moved one lane up or down; the end lane takes `end`.
template <int CTRL, typename S>
__device__ __forceinline__ S lane_move(S x, S end)
{
    S r;
    if constexpr (sizeof(S) == 8) {
        int a[2], e[2];
        __builtin_memcpy(a, &x, 8);
        __builtin_memcpy(e, &end, 8);
        a[0] = __builtin_amdgcn_update_dpp(e[0], a[0], CTRL, 0xf, 0xf, false);
        a[1] = __builtin_amdgcn_update_dpp(e[1], a[1], CTRL, 0xf, 0xf, false);
        __builtin_memcpy(&r, a, 8);
    } else {
        static_assert(sizeof(S) == 4, "4 or 8 bytes");
        int a, e;
        __builtin_memcpy(&a, &x, 4);
        __builtin_memcpy(&e, &end, 4);
        a = __builtin_amdgcn_update_dpp(e, a, CTRL, 0xf, 0xf, false);
        __builtin_memcpy(&r, &a, 4);
    }
    return r;
}
template <typename S>
__device__ __forceinline__ S lane_from_left(S x, S end) { return lane_move<0x138>(x, end); }   // wave_shr:1
template <typename S>
__device__ __forceinline__ S lane_from_right(S x, S end) { return lane_move<0x130>(x, end); }  // wave_shl:1

// Buffer accesses: loads past a descriptor's end return 0 and touch no memory,
// stores past it are dropped. The marching loop makes every access this way and
// gives threads (or rows) with nothing to move an offset past the end (or an
// empty descriptor) instead of branching: loads and stores count in one counter
// here, and a wait for the next row's loads can only let later accesses stay in
// flight if their number is the same on every way to the wait.
constexpr uint32_t NOWHERE = 0x80000000u;
using BufferRsrc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ BufferRsrc buffer_at(const void* p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// B bytes at off (per lane) + soff (uniform) into x.
template <typename T>
__device__ __forceinline__ void buffer_load(BufferRsrc b, T& x, uint32_t off, uint32_t soff)
{
    if constexpr (sizeof(T) == 16) {
        const u32x4_t r = __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, (int)soff, 0);
        __builtin_memcpy(&x, &r, 16);
    } else if constexpr (sizeof(T) == 8) {
        const u32x2_t r = __builtin_amdgcn_raw_buffer_load_b64(b, (int)off, (int)soff, 0);
        __builtin_memcpy(&x, &r, 8);
    } else if constexpr (sizeof(T) == 4) {
        const uint32_t r = __builtin_amdgcn_raw_buffer_load_b32(b, (int)off, (int)soff, 0);
        __builtin_memcpy(&x, &r, 4);
    } else {
        static_assert(sizeof(T) == 2, "2, 4, 8 or 16 bytes");
        const uint16_t r = __builtin_amdgcn_raw_buffer_load_b16(b, (int)off, (int)soff, 0);
        __builtin_memcpy(&x, &r, 2);
    }
}

// The same stored, non-temporal (NT) or plain.
template <bool NT_, typename T>
__device__ __forceinline__ void buffer_store(BufferRsrc b, const T& x, uint32_t off, uint32_t soff)
{
    constexpr int NT = NT_ ? 2 : 0;
    if constexpr (sizeof(T) == 16) {
        u32x4_t r;
        __builtin_memcpy(&r, &x, 16);
        __builtin_amdgcn_raw_buffer_store_b128(r, b, (int)off, (int)soff, NT);
    } else if constexpr (sizeof(T) == 8) {
        u32x2_t r;
        __builtin_memcpy(&r, &x, 8);
        __builtin_amdgcn_raw_buffer_store_b64(r, b, (int)off, (int)soff, NT);
    } else {
        static_assert(sizeof(T) == 4, "4, 8 or 16 bytes");
        uint32_t r;
        __builtin_memcpy(&r, &x, 4);
        __builtin_amdgcn_raw_buffer_store_b32(r, b, (int)off, (int)soff, NT);
    }
}

// Where a thread's loads of a row lie: byte offsets from one element before the
// row (columns i0 of its vectors, and the columns next to them where neither the
// vectors nor the neighbour lanes have them; at the domain's sides the column
// that stands in), or NOWHERE.
struct RowOffsets {
    uint32_t vec, left, right, mask;
};

// Issues everything a row's first step reads; nothing waits for a value here.
template <typename S, int V>
__device__ __forceinline__ void load_row(RowLoad<S, V>& d, uint32_t (&mask)[(V + 3) / 4], const S* src,
                                         const Rows3& rows, uint32_t pop_bytes, const RowOffsets& at,
                                         const uint8_t* mask_row, bool solid)
{
    constexpr uint32_t B = sizeof(S);
    struct Vec { S x[V]; };
    struct MaskBytes { uint8_t x[V]; };
    const uint32_t row_bytes = 9 * pop_bytes + 2 * B;
    const BufferRsrc row[3] = {buffer_at(src + rows.o[0] - 1, row_bytes), buffer_at(src + rows.o[1] - 1, row_bytes),
                               buffer_at(src + rows.o[2] - 1, row_bytes)};
    MaskBytes mb;
    buffer_load(buffer_at(mask_row, solid ? pop_bytes / B : 0), mb, at.mask, 0);
#pragma unroll
    for (int w = 0; w < (V + 3) / 4; ++w) mask[w] = 0;
    __builtin_memcpy(mask, &mb, V);
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        buffer_load(row[ROWQ[EXP[m]]], d.left[m], at.left, EXP[m] * pop_bytes);
        buffer_load(row[ROWQ[EXM[m]]], d.right[m], at.right, EXM[m] * pop_bytes);
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        Vec v;
        // one element off for the x-shifted directions of the vectors that load so
        const uint32_t shift = RowLoad<S, V>::kShifted ? (uint32_t)(1 - EXQ[q]) * B : B;
        buffer_load(row[ROWQ[q]], v, at.vec + shift, (uint32_t)q * pop_bytes);
        __builtin_memcpy(d.v[q], v.x, sizeof(v));
    }
}

// The loaded row with its ends in place: left and right become the neighbours of
// the thread's first and last node (vectors that shift by lane moves), and the
// domain's sides are resolved (a column past the domain is not a node: the
// neighbour of the last column is put there). west, east: the wavefront holds the
// domain's first, last column (thread index `last_col` of it, if 0 .. V - 1).
template <typename S, int V>
__device__ __forceinline__ void resolve_row(RowLoad<S, V>& d, bool west, bool east, uint32_t il, int last_col,
                                            const Sides& sd, const S (&inflow)[2][3])
{
    constexpr bool kShifted = RowLoad<S, V>::kShifted;
    if (west) {
        const int c = opaque((int)il);
        const bool me = c == 0, in_me = c == (sd.west_col < 0 ? 0 : -1);
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const S in = inflow[0][m], x = in_me ? in : d.left[m];
            if constexpr (kShifted) d.v[EXP[m]][0] = me ? x : d.v[EXP[m]][0];
            else d.left[m] = x;
        }
    }
    if constexpr (!kShifted) {
#pragma unroll
        for (int m = 0; m < 3; ++m) d.left[m] = lane_from_left(d.v[EXP[m]][V - 1], d.left[m]);
    }
    if (east) {
        const int c = opaque(last_col);
        const bool in_me = (uint32_t)c < (sd.east_col < 0 ? (uint32_t)V : 0u);
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const S in = inflow[1][m], e = in_me ? in : d.right[m];
            if constexpr (kShifted) {
#pragma unroll
                for (int k = 0; k < V; ++k) d.v[EXM[m]][k] = k == c ? e : d.v[EXM[m]][k];
            } else {
#pragma unroll
                for (int k = 1; k < V; ++k) d.v[EXM[m]][k] = k - 1 == c ? e : d.v[EXM[m]][k];
                const S x = lane_from_right(d.v[EXM[m]][0], e);
                d.right[m] = c == V - 1 ? e : x;
            }
        }
    } else if constexpr (!kShifted) {
#pragma unroll
        for (int m = 0; m < 3; ++m) d.right[m] = lane_from_right(d.v[EXM[m]][0], d.right[m]);
    }
}

template <int V>
__device__ __forceinline__ int mask_of(const uint32_t (&w)[(V + 3) / 4], int k)
{
    return (int)((w[k / 4] >> (8 * (k % 4))) & 255u);
}

// V elements of a thread's own in LDS, as one aligned access.
template <typename S, int V>
__device__ __forceinline__ void lds_vec(const S* p, S (&x)[V])
{
    __builtin_memcpy(x, __builtin_assume_aligned(p, V * sizeof(S)), V * sizeof(S));
}
template <typename S, int V>
__device__ __forceinline__ void set_lds_vec(S* p, const S (&x)[V])
{
    __builtin_memcpy(__builtin_assume_aligned(p, V * sizeof(S)), x, V * sizeof(S));
}

// The record of one tile of one step: the wavefront's mass partial and, in tiles
// holding solid nodes, a force partial per slot (the single step's partials, in
// its order); nothing is written unless `on`. lds: 2 SLOT_PASS doubles per
// wavefront.
constexpr int SLOT_PASS = 16;
template <int V, typename R>
__device__ __forceinline__ void record_tile(const KernelArgs<R>& args, bool on, int t, int buf, double drho, int s0,
                                            int s1, const uint32_t (&mask)[(V + 3) / 4], const R* fv, int n_own,
                                            double* lds)
{
    const auto* a = args.get();
    const int block = a->block, nw = block >> 6;
    double* mass_part = a->mass_part + buf * a->fin.mass_stride;
    const int lane = (int)(threadIdx.x & 63), wid = (int)threadIdx.x >> 6;
    const double wm = wave_sum_lane63(drho);
    buffer_store<true>(buffer_at(mass_part + (int64_t)t * nw, (uint32_t)nw * 8), wm,
                 on && lane == 63 ? (uint32_t)wid * 8 : NOWHERE, 0);
    if (!on || s1 <= s0) return;
    double* slot_force = a->slot_force + buf * a->fin.slot_stride;
    const int32_t* slot_body = a->slot_body;
    const int own = opaque(n_own);
#pragma unroll 1
    for (int c0 = s0; c0 < s1; c0 += SLOT_PASS) {
        const int c1 = min(s1, c0 + SLOT_PASS);
#pragma unroll 1
        for (int s = c0; s < c1; ++s) {
            const int b = table_at(slot_body, s);
            double px = 0.0, py = 0.0;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                if (k < own && mask_of<V>(mask, k) == b) {
                    px -= (double)fv[k * block + (int)threadIdx.x];
                    py -= (double)fv[(V + k) * block + (int)threadIdx.x];
                }
            }
            const double wx = wave_sum_lane63(px);
            const double wy = wave_sum_lane63(py);
            if (lane == 63) {
                lds[2 * ((s - c0) * nw + wid)] = wx;
                lds[2 * ((s - c0) * nw + wid) + 1] = wy;
            }
        }
        __syncthreads();
        for (int s = c0 + (int)threadIdx.x; s < c1; s += block) {
            double x = 0.0, y = 0.0;
            for (int w = 0; w < nw; ++w) {
                x += lds[2 * ((s - c0) * nw + w)];
                y += lds[2 * ((s - c0) * nw + w) + 1];
            }
            slot_force[2 * s] = x;
            slot_force[2 * s + 1] = y;
        }
        __syncthreads();   // lds is reused by the next batch of slots
    }
}

template <typename R>
__device__ __forceinline__ BodySource<R> mask_bodies()
{
    BodySource<R> bs;
    bs.uniform = false;
    bs.pose = nullptr;
    bs.near = 0;
    return bs;
}

// One step of a thread's V nodes: gather(k, f) gives node k's streamed
// populations; the results go to out, encoded. Returns the sum of its own nodes'
// density deviations; a solid node's force goes to fv ([2][V][block] in LDS).
template <typename S, int V, bool RECORD, typename R, typename Gather>
__device__ __forceinline__ double row_nodes(Gather gather, S (&out)[9][V], const uint32_t (&mask)[(V + 3) / 4], int i0,
                                            int j, int n_own, bool ragged, const StepArgs<R>& a, R* fv)
{
    const BodySource<R> bs = mask_bodies<R>();
    double drho = 0.0;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        R f[9];
        gather(k, f);
        const int body = mask_of<V>(mask, k);
        const NodeResult<R> n = collide_node<R, false, true>(f, body, i0 + k, j, a, bs);
#pragma unroll
        for (int q = 0; q < 9; ++q) out[q][k] = enc<S>(f[q]);
        if constexpr (RECORD) {
            if (body) {
                fv[k * a.block + (int)threadIdx.x] = n.fvx;
                fv[(V + k) * a.block + (int)threadIdx.x] = n.fvy;
            }
            R d = n.drho;
            if (ragged) d = k < opaque(n_own) ? d : R(0);
            drho += (double)d;
        }
    }
    return drho;
}

// The first step at one node (column c, row j), for the columns next to a strip:
// its populations that enter the strip (EXP on the west, EXM on the east).
template <typename S, typename R>
__device__ __forceinline__ void edge_node(const S* src, bool east, int c, int j, const StepArgs<R>& a,
                                          const Sides& sd, const S (&inflow)[2][3], S (&o)[3])
{
    const Rows3 rows = rows_of(j, a);
    R f[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        int x = c - EXQ[q];
        S v;
        if (EXQ[q] == 1) {
            if (x < 0) x = sd.west_col;
            v = side_value(src, rows.o[ROWQ[q]] + q * a.plane, x, inflow[0], q == EXP[0] ? 0 : q == EXP[1] ? 1 : 2);
        } else if (EXQ[q] == -1) {
            if (x >= a.nx) x = sd.east_col;
            v = side_value(src, rows.o[ROWQ[q]] + q * a.plane, x, inflow[1], q == EXM[0] ? 0 : q == EXM[1] ? 1 : 2);
        } else {
            v = src[rows.o[ROWQ[q]] + q * a.plane + x];
        }
        f[q] = dec(v);
    }
    const int body = a.mask[(int64_t)j * a.pitch + c];
    const BodySource<R> bs = mask_bodies<R>();
    collide_node<R, false, true>(f, body, c, j, a, bs);
#pragma unroll
    for (int m = 0; m < 3; ++m) o[m] = enc<S>(east ? f[EXM[m]] : f[EXP[m]]);
}

// A row's e_y = 0 and e_y = +1 populations into the thread's LDS slots.
template <typename S, int V>
__device__ __forceinline__ void hold_row(S* hold, S* ring, int slot, const S (&h)[9][V])
{
    set_lds_vec<S, V>(hold, h[0]);
    set_lds_vec<S, V>(hold + slot, h[1]);
    set_lds_vec<S, V>(hold + 2 * slot, h[3]);
    set_lds_vec<S, V>(ring, h[2]);
    set_lds_vec<S, V>(ring + slot, h[5]);
    set_lds_vec<S, V>(ring + 2 * slot, h[6]);
}

template <typename S, int V, bool RECORD>
__global__ void __launch_bounds__(MAX_BLOCK)
k_march(const S* __restrict__ src, S* __restrict__ dst, StepArgs<typename Arith<S>::R> a, MarchArgs m)
{
    using R = typename Arith<S>::R;
    // per thread, nine results of V nodes held for the second step (see below); the
    // blocks that sum records use it for their trees
    extern __shared__ __align__(16) unsigned char lds_dyn[];
    const int lead = a.fin_n > 0 ? N_XCD : 0;
    if ((int)blockIdx.x < lead) {
        finalize_record(a.fin, a.fin_buf, a.fin_n, (int)blockIdx.x, N_XCD, reinterpret_cast<double*>(lds_dyn));
        return;
    }
    __shared__ S edge[2][MARCH_ROWS + 2][3];      // first step next to the strip: column x0 - 1, column xe
    __shared__ S ends[2][MAX_BLOCK / 64][2][3];   // ... at the wavefronts' ends: last column, first column
    __shared__ S inflow[2][3];
    __shared__ double lds[2 * SLOT_PASS * (MAX_BLOCK / 64)];
    // each XCD takes a contiguous eighth of the (chunk, strip) pairs
    const int blk = (int)blockIdx.x - lead;
    const int id = (blk % N_XCD) * m.per_xcd + blk / N_XCD;
    if (id >= m.n_chunks * a.tiles_x) return;   // whole block
    const int chunk = uniform(id / a.tiles_x), tx = id - chunk * a.tiles_x, y0 = chunk * m.rows;
    const int n_rows = min(m.rows, a.ny - y0);
    const int lane = (int)(threadIdx.x & 63), wid = uniform((int)threadIdx.x >> 6);
    const int nw = a.block >> 6;
    const int x0 = tx * a.tile_w, xe = min(x0 + a.tile_w, a.nx);
    const uint32_t i0 = (uint32_t)(x0 + (int)threadIdx.x * V);
    const int n_own = max(0, min(V, a.nx - (int)i0));
    const uint32_t il = n_own > 0 ? i0 : 0;
    const int last = xe - 1 - (int)i0;        // this thread's index of the strip's last column, if 0 .. V - 1
    const int east = a.nx - 1 - (int)i0;      // ... and of the domain's
    const int64_t P = a.plane;
    const uint32_t pop_bytes = (uint32_t)P * (uint32_t)sizeof(S);
    const uint32_t store_off = n_own == V ? i0 * (uint32_t)sizeof(S) : NOWHERE;
    const bool ragged = a.nx - x0 < a.tile_w;   // some threads own fewer than V columns
    const bool wave_west = x0 == 0 && wid == 0, wave_east = __builtin_amdgcn_ballot_w64(east >= 0 && east < V) != 0;
    const bool wave_last = __builtin_amdgcn_ballot_w64(last >= 0 && last < V) != 0;
    const int buf2 = (a.part_buf + (m.rec & 1)) & (a.fin.n_buf - 1);
    const KernelArgs<R> args;
    if (threadIdx.x < 3) {
        const int d = (int)threadIdx.x;
        inflow[0][d] = enc<S>(d == 0 ? a.feq_in[EXP[0]] : d == 1 ? a.feq_in[EXP[1]] : a.feq_in[EXP[2]]);
        inflow[1][d] = enc<S>(d == 0 ? a.feq_in[EXM[0]] : d == 1 ? a.feq_in[EXM[1]] : a.feq_in[EXM[2]]);
    }
    __syncthreads();
    const Sides sd = {a.west == SIDE_INFLOW_EQ ? -1 : (a.west == SIDE_PERIODIC ? a.nx - 1 : 0),
                         a.east == SIDE_INFLOW_EQ ? -1 : (a.east == SIDE_PERIODIC ? 0 : a.nx - 1)};

    RowOffsets at;
    {
        constexpr uint32_t B = sizeof(S);
        constexpr bool kShifted = RowLoad<S, V>::kShifted;
        const bool at_east = east >= 0 && east < V;
        at.vec = il * B;
        at.mask = il;
        at.left = (kShifted ? il == 0 : lane == 0) ? ((il > 0 ? il - 1 : (uint32_t)max(sd.west_col, 0)) + 1) * B : NOWHERE;
        at.right = at_east ? ((uint32_t)max(sd.east_col, 0) + 1) * B
                           : (!kShifted && lane == 63 && east >= V ? (il + V + 1) * B : NOWHERE);
    }

    // the columns next to the strip, all rows of the first step; outside the
    // domain, the column that stands in for it
    for (int e = (int)threadIdx.x; e < 2 * (n_rows + 2); e += a.block) {
        const bool right = e >= n_rows + 2;
        const int k = right ? e - (n_rows + 2) : e;
        int j = y0 - 1 + k;
        j = j < 0 ? j + a.ny : (j >= a.ny ? j - a.ny : j);
        const int c = right ? (xe < a.nx ? xe : sd.east_col) : (x0 > 0 ? x0 - 1 : sd.west_col);
        S o[3];
        if (c >= 0) {
            edge_node(src, right, c, j, a, sd, inflow, o);
        } else {
#pragma unroll
            for (int d = 0; d < 3; ++d) o[d] = right ? inflow[1][d] : inflow[0][d];
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) edge[right ? 1 : 0][k][d] = o[d];
    }
    __syncthreads();

    // Row by row: pass `it` does the first step of row r = y0 - 1 + it, then the
    // second step of row r - 1, which streams from the first step's rows r - 2 (e_y =
    // +1), r - 1 (e_y = 0) and r (e_y = -1, still in h). Of the other two rows each
    // thread keeps its own V nodes' values in LDS, one vector access a population:
    // row r - 1's e_y = 0 (slots 0 .. 2) and e_y = +1 populations and row r - 2's e_y
    // = +1 ones (slots 3 .. 5 and 6 .. 8 in turn). Their end elements, from the
    // neighbour lanes when the row was new, stay in registers.
    S* hold = reinterpret_cast<S*>(lds_dyn) + (int)threadIdx.x * V;
    const int slot = a.block * V;
    R* fv = reinterpret_cast<R*>(reinterpret_cast<S*>(lds_dyn) + 9 * slot);
    S h[9][V];                            // row r's first step
    S hl[3], hr[3];                       // its columns i0 - 1 of EXP and i0 + V of EXM
    S a1l, a3r, b5l[2], b6r[2];           // those of the held rows
    uint32_t mask[(V + 3) / 4], pmask[(V + 3) / 4];   // body ids of rows r and r - 1
    int r = uniform(y0 == 0 ? a.ny - 1 : y0 - 1);
    Rows3 rows = rows_of(r, a);
    int64_t drow = (int64_t)y0 * a.lstride;       // rows y0 .. y0 + n_rows - 1 in turn: no wrap
    int s0 = 0, s1 = 0, ps0 = 0, ps1 = 0;         // force slots of rows r and r - 1; the next row's are
    int n0 = uniform(table_at(a.tile_slot_ptr, r * a.tiles_x + tx));   // read a pass ahead
    int n1 = uniform(table_at(a.tile_slot_ptr, r * a.tiles_x + tx + 1));

    // the first step of row r
    auto first = [&](int it) {
        s0 = n0;
        s1 = n1;
        RowLoad<S, V> cur;
        load_row<S, V>(cur, mask, src, rows, pop_bytes, at, a.mask + (int64_t)r * a.pitch, s1 > s0);
        const int rn = uniform(r == a.ny - 1 ? 0 : r + 1);
        n0 = table_at(a.tile_slot_ptr, rn * a.tiles_x + tx);
        n1 = table_at(a.tile_slot_ptr, rn * a.tiles_x + tx + 1);
        resolve_row<S, V>(cur, wave_west, wave_east, il, east, sd, inflow);
        auto pulled = [&](int k, R (&f)[9]) {
#pragma unroll
            for (int q = 0; q < 9; ++q) f[q] = dec(cur.v[q][k]);
            if constexpr (!RowLoad<S, V>::kShifted) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    f[EXP[d]] = dec(k == 0 ? cur.left[d] : cur.v[EXP[d]][k > 0 ? k - 1 : 0]);
                    f[EXM[d]] = dec(k == V - 1 ? cur.right[d] : cur.v[EXM[d]][k < V - 1 ? k + 1 : 0]);
                }
            }
        };
        const double drho = row_nodes<S, V, RECORD>(pulled, h, mask, (int)i0, r, n_own, ragged, a, fv);
        if constexpr (RECORD)
            record_tile<V>(args, (m.rec & 1) && it > 0 && it <= n_rows, r * a.tiles_x + tx, a.part_buf, drho, s0, s1, mask,
                           fv, n_own, lds);   // the chunk's own rows only

        // the row's end elements through LDS (double-buffered: one barrier a row)
        const int pb = it & 1;
        if (nw > 1) {
            if (lane == 63) {
#pragma unroll
                for (int d = 0; d < 3; ++d) ends[pb][wid][0][d] = h[EXP[d]][V - 1];
            }
            if (lane == 0) {
#pragma unroll
                for (int d = 0; d < 3; ++d) ends[pb][wid][1][d] = h[EXM[d]][0];
            }
            __syncthreads();
        }
        const S* wl = wid > 0 ? ends[pb][wid - 1][0] : edge[0][it];
        const S* wr = wid < nw - 1 ? ends[pb][wid + 1][1] : edge[1][it];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            hl[d] = lane_from_left(h[EXP[d]][V - 1], wl[d]);
            hr[d] = lane_from_right(h[EXM[d]][0], wr[d]);
        }
        if (wave_last) {   // the strip's last column: its neighbour is column xe
            const int c = opaque(last);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const S e = edge[1][it][d];
                hr[d] = c == V - 1 ? e : hr[d];
#pragma unroll
                for (int k = 1; k < V; ++k) h[EXM[d]][k] = k - 1 == c ? e : h[EXM[d]][k];   // past the domain
            }
        }
    };
    // the held rows move down one place, row r joins them, on to the next row
    auto next_row = [&]() {
        b5l[1] = b5l[0];
        b6r[1] = b6r[0];
        b5l[0] = hl[1];
        b6r[0] = hr[1];
        a1l = hl[0];
        a3r = hr[0];
#pragma unroll
        for (int w = 0; w < (V + 3) / 4; ++w) pmask[w] = mask[w];
        ps0 = s0;
        ps1 = s1;
        r = uniform(r == a.ny - 1 ? 0 : r + 1);
        rows.o[1] = uniform(rows.o[0]);
        rows.o[0] = uniform(rows.o[2]);
        rows.o[2] = uniform(r == a.ny - 1 ? 0 : rows.o[2] + a.lstride);
    };

#pragma unroll 1
    for (int it = 0; it < 2; ++it) {   // rows y0 - 1 and y0: nothing to stream from yet
        first(it);
        hold_row(hold, hold + (3 + 3 * (it & 1)) * slot, slot, h);
        next_row();
    }
#pragma unroll 1
    for (int it = 2; it < n_rows + 2; ++it) {
        first(it);
        // ---- second step, row r - 1 = y0 + it - 2; row r's results to LDS
        S* ring = hold + (3 + 3 * (it & 1)) * slot;   // row r - 2's e_y = +1 populations, then row r's
        S a0[V], a1[V], a3[V], b2[V], b5[V], b6[V];
        lds_vec<S, V>(hold, a0);
        lds_vec<S, V>(hold + slot, a1);
        lds_vec<S, V>(hold + 2 * slot, a3);
        lds_vec<S, V>(ring, b2);
        lds_vec<S, V>(ring + slot, b5);
        lds_vec<S, V>(ring + 2 * slot, b6);
        hold_row(hold, ring, slot, h);
        auto held = [&](int k, R (&f)[9]) {
            constexpr int L = V - 1;
            f[0] = dec(a0[k]);
            f[1] = dec(k == 0 ? a1l : a1[k > 0 ? k - 1 : 0]);
            f[3] = dec(k == L ? a3r : a3[k < L ? k + 1 : 0]);
            f[2] = dec(b2[k]);
            f[5] = dec(k == 0 ? b5l[1] : b5[k > 0 ? k - 1 : 0]);
            f[6] = dec(k == L ? b6r[1] : b6[k < L ? k + 1 : 0]);
            f[4] = dec(h[4][k]);
            f[8] = dec(k == 0 ? hl[2] : h[8][k > 0 ? k - 1 : 0]);
            f[7] = dec(k == L ? hr[2] : h[7][k < L ? k + 1 : 0]);
        };
        const int y = y0 + it - 2;
        S out[9][V];
        const double drho = row_nodes<S, V, RECORD>(held, out, pmask, (int)i0, y, n_own, ragged, a, fv);
        const BufferRsrc row = buffer_at(dst + drow, 9 * pop_bytes);
        with_hint(blk / N_XCD >= m.keep, [&](auto hint) {
            constexpr bool NT = decltype(hint)::value;
#pragma unroll
            for (int q = 0; q < 9; ++q) buffer_store<NT>(row, out[q], store_off, (uint32_t)q * pop_bytes);
        });
        if (ragged) {   // the last columns of a row that ends inside a vector
#pragma unroll
            for (int k = 0; k < V; ++k)
                if (k < opaque(n_own) && n_own < V)
#pragma unroll
                    for (int q = 0; q < 9; ++q) store_one<S, true>(at_off32(dst + (drow + q * P + k), i0), out[q][k]);
        }
        drow = uniform(drow + a.lstride);
        if constexpr (RECORD)
            record_tile<V>(args, (m.rec & 2) != 0, y * a.tiles_x + tx, buf2, drho, ps0, ps1, pmask, fv, n_own, lds);
        next_row();
    }
}

template <typename S, int V>
hipError_t march_v(const S* in, S* out, const StepArgs<typename Arith<S>::R>& a, const MarchArgs& m, hipStream_t s)
{
    const int lead = a.fin_n > 0 ? N_XCD : 0;
    const dim3 grid((unsigned)(m.per_xcd * N_XCD + lead)), block((unsigned)a.block);
    const size_t nodes = (size_t)V * (size_t)a.block;
    const size_t lds = std::max(9 * nodes * sizeof(S) + (m.rec ? 2 * nodes * sizeof(typename Arith<S>::R) : 0),
                                2 * FIN_LANES * sizeof(double));
    if (m.rec) hipLaunchKernelGGL((k_march<S, V, true>), grid, block, lds, s, in, out, a, m);
    else hipLaunchKernelGGL((k_march<S, V, false>), grid, block, lds, s, in, out, a, m);
    return hipGetLastError();
}

}  // namespace

template <typename S>
hipError_t MarchLaunch<S>::one(const void* src, void* dst, const void* step_args, const MarchArgs& m, hipStream_t s)
{
    using R = typename Arith<S>::R;
    const StepArgs<R>& a = *static_cast<const StepArgs<R>*>(step_args);
    const S* in = static_cast<const S*>(src);
    S* out = static_cast<S*>(dst);
    constexpr int VW = 16 / (int)sizeof(S);
    if (a.vec != VW) return hipErrorInvalidValue;
    return march_v<S, VW>(in, out, a, m, s);
}

}  // namespace lbvp
