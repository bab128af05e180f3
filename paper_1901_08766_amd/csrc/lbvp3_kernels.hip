// lbvp3_kernels.hip -- gfx950 kernels of the fused D3Q19 TRT-VP time step.
//
// The 3-D extension of the scheme (the paper states it on D2Q9, Sec. 2.2, and
// names 3-D as its next step, Sec. 4). Layout in HBM: lattice rows of
// structures of arrays, population a of node (i, j, k) at
//   lattice[r * lstride + a * pitch + i],  r = k * ny + j,  lstride = 19 pitch,
// so that the 19 population rows of one lattice row lie back to back and a
// tile's loads and stores stay within a few neighbouring rows of memory. pitch
// is a multiple of 64 elements. Every storage type holds the weight-normalized
// deviation h_a = (f_a - w_a rho0) / w_a; the moments use the integers
// 36 w_a = 12 (rest), 2 (faces), 1 (edges):
//   36 drho = 12 h_0 + 2 sum_faces h + sum_edges h,   36 j = sum e_a (36 w_a) h_a,
// and in these units the equilibrium is h^eq_a = drho + rho (3 eu + 9/2 eu^2 - 3/2 u.u)
// and the Guo term F_a / w_a = 3 (e_a - u).F + 9 (e_a.u)(e_a.F) (eqs. feq,
// external-force-term with the D3Q19 weights; c_s^2 = 1/3). The odd part of the
// equilibrium, 3 rho e.u, is formed as e.(36 j + 18 F)/12 from the momentum.
//
// One step per node, fused (Sec. 2.2, steps (2)-(6)):
//   pull     f_a(x) = g_a(x - e_a)                                   eq. (streaming)
//   rho = rho0 + sum w_a h_a,  u* = (j + F_b/2) / rho                eqs. (rho), (rho*velocity-star)
//   du = chi (U_O - u*) / (2 eta + chi),  F_VP = 2 rho du            eqs. (d-V), (force-density)
//   u = u* + du,  F = F_b + F_VP                                     eq. (velocity-r)
//   TRT collision of the nine (a, opposite a) pairs and the rest population with
//   the even/odd split of f^eq and of the Guo term          eqs. (TRT-collision), (collision-modified)
// with U_O = v + omega x (x - c) of the node's body.
//
// The step is bound by HBM traffic: 19 loads, 19 stores and a mask byte per node
// against ~350 flops. Each thread owns V consecutive nodes of a row and moves
// each population with one V-wide access; the directions with an x component
// load V elements one element off alignment (a single dword-aligned vector
// load), or, for 2-byte vectors, aligned with the end element from a lane shuffle.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lbvp3_internal.h"
#include "lbvp_device.h"

namespace lbvp3 {
namespace {

using lbvp::Arith;
using lbvp::as_lv;
using lbvp::at_off32;
using lbvp::collide_pair;
using lbvp::dec;
using lbvp::div36;
using lbvp::enc;
using lbvp::FIN_LANES;
using lbvp::lane_sum;
using lbvp::load_mask;
using lbvp::load_vec;
using lbvp::load_vec_shifted;
using lbvp::momentum3;
using lbvp::NodeTerms;
using lbvp::Pair;
using lbvp::recip;
using lbvp::store_one;
using lbvp::store_vec;
using lbvp::with_hint;
using lbvp::wave_sum_lane63;
using lbvp::xcd_tile;

template <typename R>
struct Node3 {
    R drho, rho, u[3], fv[3];
};

// Steps (4)-(6) at node (i, j, k) with streamed populations f (weight-normalized);
// overwrites f with the post-collision populations.
// EXACT_MOM as in the 2-D step: the 2-byte storage types take 3 rho u as (3 rho) u.
// FIELDS: the node's density, velocity and force are stored.
template <typename R, bool EXACT_MOM = true, bool FIELDS = false>
__device__ __forceinline__ Node3<R> collide3(R (&f)[Q], int body, int i, int j, int k, const Step3Args<R>& a)
{
    const R faces = ((f[1] + f[2]) + (f[3] + f[4])) + (f[5] + f[6]);
    const R edges = (((f[7] + f[8]) + (f[9] + f[10])) + ((f[11] + f[12]) + (f[13] + f[14]))) +
                    ((f[15] + f[16]) + (f[17] + f[18]));
    const R drho = div36(R(12) * f[0] + (R(2) * faces + edges));
    const R rho = a.rho0 + drho;
    const R inv_36rho = recip<FIELDS>(R(36) * rho);
    const R d78 = f[7] - f[8], d910 = f[9] - f[10], d1112 = f[11] - f[12], d1314 = f[13] - f[14];
    const R d1516 = f[15] - f[16], d1718 = f[17] - f[18];
    // 36 j from the odd parts of the pairs, plus 18 F_b (eq. rho*velocity-star)
    R j36[3], u[3];
    j36[0] = R(2) * (f[1] - f[2]) + ((d78 + d910) + (d1112 + d1314)) + a.fb18[0];
    j36[1] = R(2) * (f[3] - f[4]) + ((d78 - d910) + (d1516 + d1718)) + a.fb18[1];
    j36[2] = R(2) * (f[5] - f[6]) + ((d1112 - d1314) + (d1516 - d1718)) + a.fb18[2];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = j36[d] * inv_36rho;

    R fv[3] = {R(0), R(0), R(0)};
    if (body) {
        const R* B = a.bodies + BODY3_STRIDE * body;
        // x - c from the split centre (a centre rounded to FP32 whole would be off
        // by up to half an FP32 spacing, the same for every node of the body)
        const R rx = ((R)i - B[0]) - B[3], ry = ((R)j - B[1]) - B[4], rz = ((R)k - B[2]) - B[5];
        R uo[3];
        uo[0] = B[6] + (B[10] * rz - B[11] * ry);
        uo[1] = B[7] + (B[11] * rx - B[9] * rz);
        uo[2] = B[8] + (B[9] * ry - B[10] * rx);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const R du = a.vp_c * (uo[d] - u[d]);
            fv[d] = R(2) * rho * du;
            u[d] += du;
        }
    }
    R F[3], P[3];   // total force; 3 rho u formed from the momentum
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        F[d] = a.fb[d] + fv[d];
        if constexpr (EXACT_MOM) P[d] = momentum3(j36[d], fv[d]);
        else P[d] = (R(3) * rho) * u[d];
    }

    NodeTerms<R> n;
    const R uu = (u[0] * u[0] + u[1] * u[1]) + u[2] * u[2];
    n.A = drho - (R(1.5) * rho) * uu;
    n.rho45 = R(4.5) * rho;
    n.uF3 = R(-3) * ((u[0] * F[0] + u[1] * F[1]) + u[2] * F[2]);
    const R g0 = a.om_p * (n.A - f[0]) + f[0] + a.k_p * n.uF3;
    // pair (a, a + 1) for odd a: e_a.u and e_a.F
    const Pair<R> p1 = collide_pair(f[1], f[2], u[0], P[0], F[0], n, a);
    const Pair<R> p3 = collide_pair(f[3], f[4], u[1], P[1], F[1], n, a);
    const Pair<R> p5 = collide_pair(f[5], f[6], u[2], P[2], F[2], n, a);
    const Pair<R> p7 = collide_pair(f[7], f[8], u[0] + u[1], P[0] + P[1], F[0] + F[1], n, a);
    const Pair<R> p9 = collide_pair(f[9], f[10], u[0] - u[1], P[0] - P[1], F[0] - F[1], n, a);
    const Pair<R> p11 = collide_pair(f[11], f[12], u[0] + u[2], P[0] + P[2], F[0] + F[2], n, a);
    const Pair<R> p13 = collide_pair(f[13], f[14], u[0] - u[2], P[0] - P[2], F[0] - F[2], n, a);
    const Pair<R> p15 = collide_pair(f[15], f[16], u[1] + u[2], P[1] + P[2], F[1] + F[2], n, a);
    const Pair<R> p17 = collide_pair(f[17], f[18], u[1] - u[2], P[1] - P[2], F[1] - F[2], n, a);
    f[0] = g0;
    f[1] = p1.ga;
    f[2] = p1.gb;
    f[3] = p3.ga;
    f[4] = p3.gb;
    f[5] = p5.ga;
    f[6] = p5.gb;
    f[7] = p7.ga;
    f[8] = p7.gb;
    f[9] = p9.ga;
    f[10] = p9.gb;
    f[11] = p11.ga;
    f[12] = p11.gb;
    f[13] = p13.ga;
    f[14] = p13.gb;
    f[15] = p15.ga;
    f[16] = p15.gb;
    f[17] = p17.ga;
    f[18] = p17.gb;
    Node3<R> out;
    out.drho = drho;
    out.rho = rho;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        out.u[d] = u[d];
        out.fv[d] = fv[d];
    }
    return out;
}

// Population q of column c + shift of the lattice row at element row_off. A 32-bit
// offset is the lane's own part of the address, on a base that is the same for all
// lanes (c + row_off >= 0; a shift of -1 belongs to the base).
template <typename S, typename R>
__device__ __forceinline__ S* pop_at(S* lat, int q, int64_t row_off, int c, const Step3Args<R>& a, int shift = 0)
{
    return lat + (row_off + (int64_t)q * a.pitch + (c + shift));
}
template <typename S, typename R>
__device__ __forceinline__ S* pop_at(S* lat, int q, uint32_t row_off, int c, const Step3Args<R>& a, int shift = 0)
{
    return at_off32(lat + ((int64_t)q * a.pitch + shift), row_off + (uint32_t)c);
}

// What a boundary column (EAST: the last) pulls from the column outside the
// domain: the populations with CX = 1 of a west side, CX = -1 of an east one.
// Inflow populations are rounded to the storage type like every stored population.
template <bool EAST, typename S, typename R, typename Off>
__device__ __forceinline__ void side_column(const S* src, const Off (&src_row)[Q], const Step3Args<R>& a, S (&e)[Q])
{
    const int side = EAST ? a.east : a.west;
    constexpr int SIGN = EAST ? -1 : 1;
    if (side == LBVP_BC_INFLOW_EQ) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (CX[q] == SIGN) e[q] = enc<S>(a.feq_in[q]);
    } else {
        const int c = (EAST == (side == LBVP_BC_PERIODIC)) ? 0 : a.nx - 1;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (CX[q] == SIGN) e[q] = *pop_at(src, q, src_row[q], c, a);
    }
}

template <typename R>
__device__ __forceinline__ R* force_lds()
{
    extern __shared__ __align__(16) unsigned char lds3_dyn[];
    return reinterpret_cast<R*>(lds3_dyn);
}

// lds: three sums per slot and wavefront of a batch of slots.
constexpr int SLOT_PASS = 8;

// Tile t: tile_rows lattice rows of tile_w nodes, V consecutive nodes per thread.
// OFF32: a lattice spans fewer than 2^32 bytes, so a lane's offsets into it fit 32
// bits and every access takes a scalar base and one of nine lane offsets. With one
// node per thread the vector unit bounds the step, and the 38 64-bit addresses, the
// products they came from and two divisions were a fifth of its 556 instructions: 5
// FP16 domains in a batch 26.0 -> 23.4 us per step, FP32 192 x 104 x 104 (bound by
// memory) 50.5 -> 50.2.
template <typename S, int V, bool RECORD, bool FIELDS, bool OFF32>
__device__ __forceinline__ void step3_body(const S* __restrict__ src, S* __restrict__ dst,
                                           const Step3Args<typename Arith<S>::R>& a, int t, int part_buf,
                                           double* lds, bool nt)
{
    using R = typename Arith<S>::R;
    const int n_rows = a.ny * a.nz;
    const int ty = t / a.tiles_x, tx = t - ty * a.tiles_x;
    const int tpr = a.tile_w / V;
    // quotients by multiplication: exact for threadIdx.x < 256; at most one too large for row
    const int lr = (int)(((uint32_t)threadIdx.x * a.tpr_mul) >> 16), lc = (int)threadIdx.x - lr * tpr;
    const int row_u = ty * a.tile_rows + lr;
    const int row = min(row_u, n_rows - 1);          // rows past the grid idle (clamped for addressing)
    int k = (int)__umulhi((uint32_t)row, a.ny_mul), j = row - k * a.ny;
    if (j < 0) {
        k -= 1;
        j += a.ny;
    }
    const int i0 = tx * a.tile_w + lc * V;
    const bool act = i0 < a.nx && row_u < n_rows && lr < a.tile_rows;   // threads past the tile's rows idle
    const int n_own = act ? min(V, a.nx - i0) : 0;

    // the lattice row each direction pulls from, (y - e_y, z - e_z), as elements: y and
    // z are periodic
    using Off = typename std::conditional<OFF32, uint32_t, int64_t>::type;
    const Off ls = (Off)a.lstride, zs = (Off)a.ny * ls;
    const Off own_row = (Off)row * ls;
    const Off y_up = j == 0 ? zs - ls : (Off)0 - ls, y_down = j == a.ny - 1 ? ls - zs : ls;
    const Off z_up = k == 0 ? (Off)(a.nz - 1) * zs : (Off)0 - zs, z_down = k == a.nz - 1 ? (Off)0 - (Off)(a.nz - 1) * zs : zs;
    Off src_row[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q)
        src_row[q] = own_row + (CY[q] == 1 ? y_up : (CY[q] == -1 ? y_down : (Off)0)) +
                     (CZ[q] == 1 ? z_up : (CZ[q] == -1 ? z_down : (Off)0));
    const int64_t r0 = (int64_t)row * a.pitch;       // mask and fields

    // this tile's (tile, body) force slots, asked for first; a tile without slots
    // holds no solid node and reads no mask
    const int s0 = a.tile_slot_ptr[t];
    const int s1 = a.tile_slot_ptr[t + 1];
    // Dword-or-wider elements (and single nodes) fetch the x-shifted directions
    // as one vector access one element off alignment. 2-byte vectors load aligned
    // and take the missing end element from the neighbouring lane (lanes that
    // start or end a wavefront or a tile row load it themselves), keeping the
    // loaded values packed in the storage type until each node's collision.
    constexpr bool kShifted = sizeof(S) >= 4 || V == 1;
    using LV = typename std::conditional<kShifted, R, S>::type;
    const int lane = (int)(threadIdx.x & 63);
    int body[V];
    double tile_drho = 0.0;
    // a wavefront without a node only takes its part in the record: with 256 threads
    // and rows of 192 nodes, one of four
    if (__builtin_amdgcn_ballot_w64(act) != 0) {
        LV v[Q][V];
        // Threads without a node of their own load column 0 of their (clamped) row
        // instead: every access stays inside the lattice, and their results are never
        // stored, summed or shuffled into an owned node.
        const int il = act ? i0 : 0;
        const int last = a.nx - 1 - i0;   // this thread's index of the last column, if 0 .. V - 1
        // As in the 2-D step, everything is requested before anything is waited for:
        // the columns next to a thread's own (in the storage type), the rows, then
        // what depends on the slots.
        const bool first_lane = kShifted ? i0 == 0 : (lane == 0 || lc == 0);
        const bool last_lane = (!kShifted && (lane == 63 || lc == tpr - 1)) || last < V;
        S left[Q], right[Q];
        if (act && first_lane) {
            if (!kShifted && i0 > 0) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (CX[q] == 1) left[q] = *pop_at(src, q, src_row[q], i0 - 1, a);
            } else {
                side_column<false>(src, src_row, a, left);
            }
        }
        if (act && last_lane) {
            if (!kShifted && last >= V) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (CX[q] == -1) right[q] = *pop_at(src, q, src_row[q], i0 + V, a);
            } else {
                side_column<true>(src, src_row, a, right);
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            S raw[V];
            if constexpr (kShifted) {
                const S* p = pop_at(src, q, src_row[q], il, a, -CX[q]);
                if (CX[q] != 0) load_vec_shifted<S, V>(p, raw);
                else load_vec<S, V>(p, raw);
            } else {
                load_vec<S, V>(pop_at(src, q, src_row[q], il, a), raw);
            }
#pragma unroll
            for (int e = 0; e < V; ++e) v[q][e] = as_lv<LV>(raw[e]);
        }
        if (s1 > s0) {
            load_mask<V>(a.mask + r0 + il, body);
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e) body[e] = 0;
        }

        // the columns next to the thread's own, put where the nodes below take them
        R from_left[Q], from_right[Q];
        if constexpr (!kShifted) {
            if (last < V - 1) {   // a row that ends inside the vector
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (CX[q] == -1)
#pragma unroll
                        for (int e = 1; e < V; ++e) v[q][e] = e - 1 == last ? right[q] : v[q][e];
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (CX[q] == 1) {
                    const R l = __shfl_up(dec(v[q][V - 1]), 1, 64);
                    from_left[q] = first_lane ? dec(left[q]) : l;
                }
                if (CX[q] == -1) {
                    const R r = __shfl_down(dec(v[q][0]), 1, 64);
                    from_right[q] = last_lane ? dec(right[q]) : r;
                }
            }
        } else {
            if (first_lane) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (CX[q] == 1) v[q][0] = as_lv<LV>(left[q]);
            }
            if (last_lane) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (CX[q] == -1)
#pragma unroll
                        for (int e = 0; e < V; ++e) v[q][e] = e == last ? as_lv<LV>(right[q]) : v[q][e];
            }
        }

        R fl[7][V];
        S out[Q][V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
            R f[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if constexpr (kShifted) {
                    f[q] = v[q][e];
                } else {
                    if (CX[q] == 1) f[q] = (e == 0) ? from_left[q] : dec(v[q][e > 0 ? e - 1 : 0]);
                    else if (CX[q] == -1) f[q] = (e == V - 1) ? from_right[q] : dec(v[q][e < V - 1 ? e + 1 : 0]);
                    else f[q] = dec(v[q][e]);
                }
            }
            const int i = i0 + e;
            const Node3<R> n = collide3<R, (sizeof(S) >= 4), FIELDS>(f, body[e], i, j, k, a);
#pragma unroll
            for (int q = 0; q < Q; ++q) out[q][e] = enc<S>(f[q]);
            fl[0][e] = n.rho;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                fl[1 + d][e] = n.u[d];
                fl[4 + d][e] = n.fv[d];
            }
            if constexpr (RECORD) {
                // the penalization force of every node of a tile holding solid nodes
                // goes to LDS at once, summed per body after the stores
                if (s1 > s0) {
                    R* fv = force_lds<R>();
#pragma unroll
                    for (int c = 0; c < 3; ++c) fv[(c * V + e) * (int)blockDim.x + (int)threadIdx.x] = n.fv[c];
                }
            }
            if (e < n_own) tile_drho += (double)n.drho;
        }

        with_hint(nt, [&](auto hint) {
            constexpr bool NT = decltype(hint)::value;
            if (n_own == V) {
#pragma unroll
                for (int q = 0; q < Q; ++q) store_vec<S, V, NT>(pop_at(dst, q, own_row, i0, a), out[q]);
            } else if (n_own > 0) {   // the ragged end of a row
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (e < n_own)
#pragma unroll
                        for (int q = 0; q < Q; ++q) store_one<S, NT>(pop_at(dst, q, own_row, i0 + e, a), out[q][e]);
            }
        });

        if constexpr (FIELDS) {
            R* fb = a.fields + r0 + i0;
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (e < n_own)
#pragma unroll
                    for (int c = 0; c < 7; ++c) fb[c * a.plane_f + e] = fl[c][e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) body[e] = 0;
    }

    if constexpr (RECORD) {
        // mass: one partial per wavefront (DPP moves only, no block barrier)
        const double wm = wave_sum_lane63(tile_drho);
        double* mass_part = a.mass_part + part_buf * a.fin.mass_stride;
        double* slot_force = a.slot_force + part_buf * a.fin.slot_stride;
        if (lane == 63) mass_part[(int64_t)t * (a.block >> 6) + (threadIdx.x >> 6)] = wm;
        // forces: only tiles that hold solid nodes (uniform across the block); each
        // slot's wavefront sums meet in LDS, a batch of slots per barrier, and are
        // added in wavefront order
        const R* fv = force_lds<R>();
        const int block = (int)blockDim.x, nw = block >> 6, wid = (int)threadIdx.x >> 6;
        for (int c0 = s0; c0 < s1; c0 += SLOT_PASS) {
            const int c1 = min(s1, c0 + SLOT_PASS);
            for (int s = c0; s < c1; ++s) {
                const int b = a.slot_body[s];
                double p[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (e < n_own && body[e] == b)
#pragma unroll
                        for (int c = 0; c < 3; ++c) p[c] -= (double)fv[(c * V + e) * block + (int)threadIdx.x];
#pragma unroll
                for (int off = 32; off > 0; off >>= 1)
#pragma unroll
                    for (int c = 0; c < 3; ++c) p[c] += __shfl_down(p[c], off, 64);
                if (lane == 0)
#pragma unroll
                    for (int c = 0; c < 3; ++c) lds[(3 * (s - c0) + c) * nw + wid] = p[c];
            }
            __syncthreads();
            for (int i = (int)threadIdx.x; i < 3 * (c1 - c0); i += block) {
                double x = lds[i * nw];
                for (int w = 1; w < nw; ++w) x += lds[i * nw + w];
                slot_force[3 * c0 + i] = x;
            }
            __syncthreads();   // lds is reused by the next batch of slots
        }
    }
}

// One wavefront sums slice `part` of a record's partials into its stage row:
// mass, then the force on each body (one pass over the slice's slots serves
// three components). The order is fixed by the partials alone, so neither the
// launch that runs it nor the way steps are split over calls changes a record by
// one bit: FIN_LANES virtual lanes (thread l takes lanes l, l + 64, l + 128,
// l + 192) meet pairwise with halving spans, two levels in the thread and six by
// lane moves. The thread's lanes are taken one after the other (in the tree's
// order 0, 2, 1, 3, each pair added when complete), so that the sums need no
// more registers than the step that the kernel is for.
__device__ __forceinline__ void slice_sums(const Fin3Args& f, int buf, int part, double* row)
{
    static_assert(FIN_LANES == 256, "four virtual lanes per thread");
    const double* pm = f.mass_part + buf * f.mass_stride;
    const double* sf = f.slot_force + buf * f.slot_stride;
    const int l = (int)(threadIdx.x & 63);
    const int m0 = (int)((int64_t)f.n_mass * part / N_SLICES), m1 = (int)((int64_t)f.n_mass * (part + 1) / N_SLICES);
    for (int b = -1; b < f.n_bodies; ++b) {   // -1: the mass
        int a0 = 0, a1 = 0;
        if (b >= 0) {
            const int s0 = f.body_slot_ptr[b], n = f.body_slot_ptr[b + 1] - s0;
            a0 = s0 + (int)((int64_t)n * part / N_SLICES);
            a1 = s0 + (int)((int64_t)n * (part + 1) / N_SLICES);
        }
        double v[3] = {0.0, 0.0, 0.0}, pair[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const int lane = l + 64 * ((i >> 1) + 2 * (i & 1));
            double y[3] = {0.0, 0.0, 0.0};
            if (b < 0) {
                y[0] = lane_sum(pm + m0, m1 - m0, lane);
            } else {
                for (int kk = a0 + lane; kk < a1; kk += FIN_LANES) {
                    const double* p = sf + 3 * f.body_slots[kk];
#pragma unroll
                    for (int c = 0; c < 3; ++c) y[c] += p[c];
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                pair[c] = (i & 1) ? pair[c] + y[c] : y[c];
                if (i & 1) v[c] = i == 1 ? pair[c] : v[c] + pair[c];
            }
        }
#pragma unroll
        for (int w = 32; w > 0; w >>= 1)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] += __shfl_down(v[c], w, 64);
        if (l == 0) {
            if (b < 0) {
                row[0] = v[0];
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c) row[1 + 3 * b + c] = v[c];
            }
        }
    }
}

// One block adds a stage buffer's rows in slice order into ring slot r, a column
// per thread (its rows are fetched at once, then added in order).
__device__ __forceinline__ void add_rows(const Fin3Args& f, const double* stage, int64_t r)
{
    const int row_len = 1 + 3 * f.max_bodies;
    for (int col = (int)threadIdx.x; col < 1 + 3 * f.n_bodies; col += (int)blockDim.x) {
        double y[N_SLICES];
#pragma unroll
        for (int p = 0; p < N_SLICES; ++p) y[p] = stage[(int64_t)p * row_len + col];
        double x = 0.0;
#pragma unroll
        for (int p = 0; p < N_SLICES; ++p) x += y[p];
        if (col == 0) f.ring_mass[r] = f.mass_offset + x;
        else f.ring_force[(r * f.max_bodies + (col - 1) / 3) * 3 + (col - 1) % 3] = x;
    }
}

// Leading blocks of a step launch. The record of the previous step: wavefront w of
// block blk sums slice blk * waves + w. The one before it: its rows are added.
// Spreading the two stages over two launches needs no fence or counter inside a
// launch; with one block per batch member doing all slices in turn, the sums
// outlasted the step of small members (5 FP16 domains of 1.5 M nodes in all in
// 64-thread blocks: 121 us a step).
__device__ __forceinline__ void lead_slices(const Fin3Args& f, int buf, int stage, int blk)
{
    const int part = blk * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6);
    if (part < N_SLICES) slice_sums(f, buf, part, f.stage[stage] + (int64_t)part * (1 + 3 * f.max_bodies));
}

__device__ __forceinline__ void lead_add(const Fin3Args& f, int stage)
{
    const int64_t count = *f.rec_count;
    add_rows(f, f.stage[stage], count % f.capacity);
    __syncthreads();   // every thread has read the count
    if (threadIdx.x == 0) *f.rec_count = count + 1;
}

// What a run leaves to sum (launch_finalize3): block blk of
// N_SLICES / FIN_BLOCK_WAVES. The last block to arrive sees every row and adds
// both records.
__device__ __forceinline__ void finalize_run(const Fin3Args& f, int buf, int stage, int add_stage, int blk, int* flag)
{
    if (buf < 0) {   // only rows to add
        if (blk == 0 && add_stage >= 0) lead_add(f, add_stage);
        return;
    }
    lead_slices(f, buf, stage, blk);
    __threadfence();   // publish the rows before counting in
    __syncthreads();
    if (threadIdx.x == 0)
        *flag = atomicAdd(reinterpret_cast<unsigned long long*>(f.arrivals), 1ull) ==
                (unsigned long long)(N_SLICES / FIN_BLOCK_WAVES - 1);
    __syncthreads();
    if (!*flag) return;
    __threadfence();   // the other blocks' rows are visible from here on
    int64_t count = *f.rec_count;
    if (add_stage >= 0) add_rows(f, f.stage[add_stage], count++ % f.capacity);
    add_rows(f, f.stage[stage], count % f.capacity);
    __syncthreads();   // every thread has read the count
    if (threadIdx.x == 0) {
        *f.rec_count = count + 1;
        *f.arrivals = 0;
    }
}

// Most wavefronts per SIMD of a step kernel. With one node per thread FP32 could run 6
// or 7 and FP64 5; grids bound by memory lose less to each other's rows with 5 and 4, us
// per step with and without the limit: FP32 512 x 256 x 256 852 and 863, 256 x 128 x 128
// 109.2 and 110.6, 192 x 104 x 104 50.3 and 50.7; FP64 1707 and 1746, 218.6 and 223, 115.1
// and 116.4, down to 144 x 72 x 72 42.0 and 43.0, and no difference below; batches of 20
// domains FP64 339 and 344, of 5 88.6 and 90.4, FP32 176 and 176, 39 and 41. A single
// FP32 domain that the last-level cache holds is not bound by memory, and its few
// rounds of blocks fill the chip better without the limit (WITHIN_CACHE): 144 x 72 x 72
// 20.7 and 20.1, 160 x 80 x 80 25.8 and 25.4, 128 x 64 x 64 14.7 and 14.6, 176 x 90 x 90
// 34.6 and 34.7. The 2-byte types, bound by the vector unit, keep what the registers
// allow (5 domains 23.4 us, 24.1 with 5).
template <typename S, int V, bool WITHIN_CACHE>
constexpr int MOST_WAVES = sizeof(S) == 8 && V == 1 ? 4 : sizeof(S) == 4 && V == 1 && !WITHIN_CACHE ? 5 : 8;

// ... and the least it has to leave registers for. The 4-node form of the 2-byte types,
// its loads all in flight, would take 4 registers more than 3 wavefronts have: with 2, us
// per recorded step against 3, FP16 256 x 128 x 128 62.5 and 57.5, 384 x 160 x 160 170
// and 142, 640 x 200 x 200 501 and 385, 800 x 300 x 300 1150 and 1003, 512 x 256 x 256
// 440 and 431 (but 500 x 250 x 250 428 and 455); batches of 8 domains 37.6 and 35.3, of 64
// 316 and 310. The form that keeps the fields would spill 11 and stays at 2.
template <typename S, int V, bool FIELDS>
constexpr int LEAST_WAVES = sizeof(S) == 2 && V == 4 && !FIELDS ? 3 : 1;

// A step launch, behind the leading blocks that sum earlier records.
template <typename S, int V, bool RECORD, bool FIELDS, bool OFF32, bool WITHIN_CACHE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((LEAST_WAVES<S, V, FIELDS>), MOST_WAVES<S, V, WITHIN_CACHE>)))
k_step3(const S* __restrict__ src, S* __restrict__ dst, Step3Args<typename Arith<S>::R> a)
{
    __shared__ double lds[3 * SLOT_PASS * 4];
    const int n_fin = a.fin_buf >= 0 ? slice_blocks(1, a.block) : 0;
    const int lead = n_fin + (a.add_stage >= 0 ? N_XCD : 0);
    if ((int)blockIdx.x < lead) {
        if ((int)blockIdx.x < n_fin) lead_slices(a.fin, a.fin_buf, a.fin_stage, (int)blockIdx.x);
        else if ((int)blockIdx.x == n_fin) lead_add(a.fin, a.add_stage);
        return;
    }
    const int t = xcd_tile(a.tiles_per_xcd, a.band_log2, lead);
    if (t >= a.n_tiles) return;   // whole block
    step3_body<S, V, RECORD, FIELDS, OFF32>(src, dst, a, t, a.part_buf, lds, ((int)blockIdx.x - lead) / N_XCD >= a.keep_tiles);
}

// Many domains in one launch: block -> (member, tile) through the tile map; each
// member's arguments and lattices live in device memory. The members step in
// lockstep: one step kind, record flag and partial buffer for all; leading
// blocks sum the members' earlier records.
template <typename S, int V, bool RECORD, bool FIELDS, bool OFF32>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((LEAST_WAVES<S, V, FIELDS>), MOST_WAVES<S, V, false>)))
k_step3_batch(Batch3Launch b)
{
    using R = typename Arith<S>::R;
    __shared__ double lds[3 * SLOT_PASS * 4];
    const Member3<R>* m = static_cast<const Member3<R>*>(b.members);
    if ((int)blockIdx.x < b.n_fin + b.n_add) {
        const int blk = (int)blockIdx.x;
        if (blk < b.n_fin) {
            const int per = N_SLICES / (int)(blockDim.x >> 6), d = blk / per;
            if (d < b.n_members) lead_slices(m[d].a.fin, b.fin_buf, b.fin_stage, blk - d * per);
        } else if (blk - b.n_fin < b.n_members) {
            lead_add(m[blk - b.n_fin].a.fin, b.add_stage);
        }
        return;
    }
    const int g = xcd_tile(b.tiles_per_xcd, b.band_log2, b.n_fin + b.n_add);
    if (g >= b.total_tiles) return;   // whole block
#if defined(__HIP_DEVICE_COMPILE__)
    // the tile map and the members do not change during a launch: read through
    // the constant address space (scalar loads no store of the step can alias),
    // the member copied once, up front
    using CI = const __attribute__((address_space(4))) int32_t;
    using CM = const __attribute__((address_space(4))) Member3<R>;
    const int d = ((CI*)b.tile_domain)[g];
    const Member3<R> md = ((CM*)m)[d];
    const int t = g - ((CI*)b.tile_start)[d];
#else
    const int d = b.tile_domain[g];
    const Member3<R>& md = m[d];
    const int t = g - b.tile_start[d];
#endif
    const int cur = md.cur ^ b.flip;
    const S* src = static_cast<const S*>(cur ? md.lat1 : md.lat0);
    S* dst = static_cast<S*>(cur ? md.lat0 : md.lat1);
    step3_body<S, V, RECORD, FIELDS, OFF32>(src, dst, md.a, t, b.part_buf, lds,
                                     ((int)blockIdx.x - b.n_fin - b.n_add) / N_XCD >= b.keep_tiles);
}

// The last records of an lbvp3_batch_step call.
template <typename R>
__global__ void __launch_bounds__(64 * FIN_BLOCK_WAVES) k_finalize3_members(Batch3Launch b)
{
    __shared__ int last;
    const Member3<R>* m = static_cast<const Member3<R>*>(b.members);
    constexpr int per = N_SLICES / FIN_BLOCK_WAVES;
    const int d = (int)blockIdx.x / per;
    finalize_run(m[d].a.fin, b.fin_buf, b.fin_stage, b.add_stage, (int)blockIdx.x - d * per, &last);
}

// The last records of an lbvp3_step call.
__global__ void __launch_bounds__(64 * FIN_BLOCK_WAVES) k_finalize3(Fin3Args f, int32_t buf, int32_t stage,
                                                                    int32_t add_stage)
{
    __shared__ int last;
    finalize_run(f, buf, stage, add_stage, (int)blockIdx.x, &last);
}

// ------------------------------------------------------------ conversions --
__constant__ double W3[Q] = {1.0 / 3.0,
                             1.0 / 18.0, 1.0 / 18.0, 1.0 / 18.0, 1.0 / 18.0, 1.0 / 18.0, 1.0 / 18.0,
                             1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0,
                             1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0};

__device__ __forceinline__ void conv_node(const Conv3Args& a, int64_t n, int64_t& lat_off, int64_t& fld_off)
{
    const int64_t per_plane = (int64_t)a.ny * a.nx;
    const int kl = (int)(n / per_plane);
    const int64_t rem = n - kl * per_plane;
    const int j = (int)(rem / a.nx), i = (int)(rem - (int64_t)j * a.nx);
    const int64_t row = (int64_t)(a.plane0 + kl) * a.ny + j;
    lat_off = row * a.lstride + i;
    fld_off = row * a.pitch + i;
}

// Algorithm step (1): equilibrium populations (eq. feq) of staged planes, in
// FP64, stored as normalized deviations; the fields of step 0 are (rho, u, 0).
template <typename S>
__global__ void __launch_bounds__(256) k_init3(S* lat, typename Arith<S>::R* fields, Conv3Args a)
{
    using R = typename Arith<S>::R;
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (int64_t)a.planes * a.ny * a.nx) return;
    int64_t lo, fo;
    conv_node(a, n, lo, fo);
    const double rho = a.rho ? a.rho[n] : a.rho0;
    double u[3];
    for (int d = 0; d < 3; ++d) u[d] = a.u[d] ? a.u[d][n] : 0.0;
    const double uu = (u[0] * u[0] + u[1] * u[1]) + u[2] * u[2];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const double eu = (CX[q] * u[0] + CY[q] * u[1]) + CZ[q] * u[2];
        const double h = (rho - a.rho0) + rho * (3.0 * eu + 4.5 * eu * eu - 1.5 * uu);
        lat[lo + q * a.pitch] = enc<S>((R)h);
    }
    if (fields) {
        fields[fo] = (R)rho;
        for (int d = 0; d < 3; ++d) {
            fields[(1 + d) * a.plane_f + fo] = (R)u[d];
            fields[(4 + d) * a.plane_f + fo] = R(0);
        }
    }
}

template <typename S>
__global__ void __launch_bounds__(256) k_decode3(const S* lat, Conv3Args a)
{
    const int64_t N = (int64_t)a.planes * a.ny * a.nx;
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    int64_t lo, fo;
    conv_node(a, n, lo, fo);
    for (int q = 0; q < Q; ++q) a.pops[q * N + n] = W3[q] * ((double)dec(lat[lo + q * a.pitch]) + a.rho0);
}

template <typename S>
__global__ void __launch_bounds__(256) k_encode3(S* lat, Conv3Args a)
{
    using R = typename Arith<S>::R;
    const int64_t N = (int64_t)a.planes * a.ny * a.nx;
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    int64_t lo, fo;
    conv_node(a, n, lo, fo);
    for (int q = 0; q < Q; ++q) lat[lo + q * a.pitch] = enc<S>((R)(a.pops[q * N + n] / W3[q] - a.rho0));
}

__global__ void k_zero_i64(int64_t* p) { *p = 0; }

template <typename S, int V, bool OFF32, bool WITHIN_CACHE>
hipError_t step_off(bool record, bool fields, const S* in, S* out, const Step3Args<typename Arith<S>::R>& a,
                    hipStream_t s)
{
    using R = typename Arith<S>::R;
    const int lead = (a.fin_buf >= 0 ? slice_blocks(1, a.block) : 0) + (a.add_stage >= 0 ? N_XCD : 0);
    const dim3 grid((unsigned)(a.tiles_per_xcd * N_XCD + lead)), block((unsigned)a.block);
    const size_t lds = record ? 3 * (size_t)V * (size_t)a.block * sizeof(R) : 0;
    if (record) {
        if (fields) hipLaunchKernelGGL((k_step3<S, V, true, true, OFF32, WITHIN_CACHE>), grid, block, lds, s, in, out, a);
        else hipLaunchKernelGGL((k_step3<S, V, true, false, OFF32, WITHIN_CACHE>), grid, block, lds, s, in, out, a);
    } else {
        if (fields) hipLaunchKernelGGL((k_step3<S, V, false, true, OFF32, WITHIN_CACHE>), grid, block, 0, s, in, out, a);
        else hipLaunchKernelGGL((k_step3<S, V, false, false, OFF32, WITHIN_CACHE>), grid, block, 0, s, in, out, a);
    }
    return hipGetLastError();
}

template <typename S, int V>
hipError_t step_v(bool record, bool fields, const S* in, S* out, const Step3Args<typename Arith<S>::R>& a,
                  hipStream_t s)
{
    if constexpr (sizeof(S) == 4 && V == 1) {
        if (a.off32 && a.keep_tiles >= a.tiles_per_xcd) return step_off<S, V, true, true>(record, fields, in, out, a, s);
    }
    return a.off32 ? step_off<S, V, true, false>(record, fields, in, out, a, s)
                   : step_off<S, V, false, false>(record, fields, in, out, a, s);
}

template <typename S>
hipError_t step_typed(bool record, bool fields, const void* src, void* dst, const void* args_v, hipStream_t s)
{
    using R = typename Arith<S>::R;
    const Step3Args<R>& a = *static_cast<const Step3Args<R>*>(args_v);
    const S* in = static_cast<const S*>(src);
    S* out = static_cast<S*>(dst);
    if (a.vec == 1) return step_v<S, 1>(record, fields, in, out, a, s);
    if constexpr (sizeof(S) >= 4) {
        if (a.vec == 2) return step_v<S, 2>(record, fields, in, out, a, s);
    }
    if constexpr (sizeof(S) == 4) {
        if (a.vec == 4) return step_v<S, 4>(record, fields, in, out, a, s);
    }
    if constexpr (sizeof(S) == 2) {   // lane-shuffle forms: 8 and 16 bytes per thread
        if (a.vec == 4) return step_v<S, 4>(record, fields, in, out, a, s);
        if (a.vec == 8) return step_v<S, 8>(record, fields, in, out, a, s);
    }
    return hipErrorInvalidValue;
}

template <typename S, int V, bool OFF32>
hipError_t batch_off(bool record, bool fields, const Batch3Launch& b, int32_t block, hipStream_t s)
{
    using R = typename Arith<S>::R;
    const dim3 grid((unsigned)(b.tiles_per_xcd * N_XCD + b.n_fin + b.n_add)), blk((unsigned)block);
    const size_t lds = record ? 3 * (size_t)V * (size_t)block * sizeof(R) : 0;
    if (record) {
        if (fields) hipLaunchKernelGGL((k_step3_batch<S, V, true, true, OFF32>), grid, blk, lds, s, b);
        else hipLaunchKernelGGL((k_step3_batch<S, V, true, false, OFF32>), grid, blk, lds, s, b);
    } else {
        if (fields) hipLaunchKernelGGL((k_step3_batch<S, V, false, true, OFF32>), grid, blk, 0, s, b);
        else hipLaunchKernelGGL((k_step3_batch<S, V, false, false, OFF32>), grid, blk, 0, s, b);
    }
    return hipGetLastError();
}

template <typename S, int V>
hipError_t batch_v(bool record, bool fields, const Batch3Launch& b, int32_t block, hipStream_t s)
{
    return b.off32 ? batch_off<S, V, true>(record, fields, b, block, s)
                   : batch_off<S, V, false>(record, fields, b, block, s);
}

template <typename S>
hipError_t batch_typed(int32_t vec, int32_t block, bool record, bool fields, const Batch3Launch& b, hipStream_t s)
{
    if (vec == 1) return batch_v<S, 1>(record, fields, b, block, s);
    if constexpr (sizeof(S) >= 4) {
        if (vec == 2) return batch_v<S, 2>(record, fields, b, block, s);
    }
    if constexpr (sizeof(S) == 4) {
        if (vec == 4) return batch_v<S, 4>(record, fields, b, block, s);
    }
    if constexpr (sizeof(S) == 2) {
        if (vec == 4) return batch_v<S, 4>(record, fields, b, block, s);
        if (vec == 8) return batch_v<S, 8>(record, fields, b, block, s);
    }
    return hipErrorInvalidValue;
}

unsigned conv_blocks(const Conv3Args& a) { return (unsigned)(((int64_t)a.planes * a.ny * a.nx + 255) / 256); }

}  // namespace

bool vec_supported(int32_t storage, int32_t vec)
{
    switch (storage) {
    case LBVP_F64: return vec == 1 || vec == 2;
    case LBVP_F32: return vec == 1 || vec == 2 || vec == 4;
    case LBVP_F16_DEV:
    case LBVP_BF16_DEV: return vec == 1 || vec == 4 || vec == 8;
    default: return false;
    }
}

hipError_t launch_step3(int32_t storage, bool record, bool fields, const void* src, void* dst, const void* step_args,
                        hipStream_t s)
{
    switch (storage) {
    case LBVP_F64: return step_typed<double>(record, fields, src, dst, step_args, s);
    case LBVP_F32: return step_typed<float>(record, fields, src, dst, step_args, s);
    case LBVP_F16_DEV: return step_typed<_Float16>(record, fields, src, dst, step_args, s);
    case LBVP_BF16_DEV: return step_typed<__bf16>(record, fields, src, dst, step_args, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step3_batch(int32_t storage, int32_t vec, int32_t block, bool record, bool fields,
                              const Batch3Launch& b, hipStream_t s)
{
    switch (storage) {
    case LBVP_F64: return batch_typed<double>(vec, block, record, fields, b, s);
    case LBVP_F32: return batch_typed<float>(vec, block, record, fields, b, s);
    case LBVP_F16_DEV: return batch_typed<_Float16>(vec, block, record, fields, b, s);
    case LBVP_BF16_DEV: return batch_typed<__bf16>(vec, block, record, fields, b, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_finalize3_members(int32_t storage, const Batch3Launch& b, hipStream_t s)
{
    const dim3 grid((unsigned)(b.n_members * (N_SLICES / FIN_BLOCK_WAVES))), block(64 * FIN_BLOCK_WAVES);
    if (storage == LBVP_F64) hipLaunchKernelGGL(k_finalize3_members<double>, grid, block, 0, s, b);
    else hipLaunchKernelGGL(k_finalize3_members<float>, grid, block, 0, s, b);
    return hipGetLastError();
}

hipError_t launch_finalize3(const Fin3Args& a, int32_t buf, int32_t stage, int32_t add_stage, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize3, dim3(N_SLICES / FIN_BLOCK_WAVES), dim3(64 * FIN_BLOCK_WAVES), 0, s, a, buf, stage,
                       add_stage);
    return hipGetLastError();
}

hipError_t launch_init3(int32_t storage, void* lat, void* fields, const Conv3Args& a, hipStream_t s)
{
    const dim3 g(conv_blocks(a)), b(256);
    switch (storage) {
    case LBVP_F64: hipLaunchKernelGGL(k_init3<double>, g, b, 0, s, (double*)lat, (double*)fields, a); break;
    case LBVP_F32: hipLaunchKernelGGL(k_init3<float>, g, b, 0, s, (float*)lat, (float*)fields, a); break;
    case LBVP_F16_DEV: hipLaunchKernelGGL(k_init3<_Float16>, g, b, 0, s, (_Float16*)lat, (float*)fields, a); break;
    case LBVP_BF16_DEV: hipLaunchKernelGGL(k_init3<__bf16>, g, b, 0, s, (__bf16*)lat, (float*)fields, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_decode3(int32_t storage, const void* lat, const Conv3Args& a, hipStream_t s)
{
    const dim3 g(conv_blocks(a)), b(256);
    switch (storage) {
    case LBVP_F64: hipLaunchKernelGGL(k_decode3<double>, g, b, 0, s, (const double*)lat, a); break;
    case LBVP_F32: hipLaunchKernelGGL(k_decode3<float>, g, b, 0, s, (const float*)lat, a); break;
    case LBVP_F16_DEV: hipLaunchKernelGGL(k_decode3<_Float16>, g, b, 0, s, (const _Float16*)lat, a); break;
    case LBVP_BF16_DEV: hipLaunchKernelGGL(k_decode3<__bf16>, g, b, 0, s, (const __bf16*)lat, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_encode3(int32_t storage, void* lat, const Conv3Args& a, hipStream_t s)
{
    const dim3 g(conv_blocks(a)), b(256);
    switch (storage) {
    case LBVP_F64: hipLaunchKernelGGL(k_encode3<double>, g, b, 0, s, (double*)lat, a); break;
    case LBVP_F32: hipLaunchKernelGGL(k_encode3<float>, g, b, 0, s, (float*)lat, a); break;
    case LBVP_F16_DEV: hipLaunchKernelGGL(k_encode3<_Float16>, g, b, 0, s, (_Float16*)lat, a); break;
    case LBVP_BF16_DEV: hipLaunchKernelGGL(k_encode3<__bf16>, g, b, 0, s, (__bf16*)lat, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_zero_i64(int64_t* p, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_i64, dim3(1), dim3(1), 0, s, p);
    return hipGetLastError();
}

}  // namespace lbvp3
