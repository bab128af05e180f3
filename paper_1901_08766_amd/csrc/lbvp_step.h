// lbvp_step.h -- gfx950 kernels of the fused D2Q9 TRT-VP time step, instantiated
// per storage type by lbvp_step_f64.hip, lbvp_step_f32.hip, lbvp_step_f16.hip and
// lbvp_step_bf16.hip.
//
// Data layout in HBM (rows of structures of arrays): population a of node (i, j)
// lives at lattice[j * lstride + a * plane + i] with plane = pitch and
// lstride = 9 pitch: the nine population rows of a lattice row lie back to back.
// pitch is a multiple of 64 elements, so every population row starts on a
// 128-byte (2-byte types) or 256-byte boundary. A tile's loads and stores then
// stay within a few neighbouring lattice rows of memory instead of touching
// nine planes a whole domain apart, which HBM serves measurably faster. All storage types hold the
// weight-normalized deviation h_a = (f_a - w_a rho0) / w_a. Its size is set by
// the flow (|h| ~ 3|u|) and is the same for every direction, and the equilibrium
// in these units carries no weight at all,
//   h^eq_a = drho + rho (3 eu + 9/2 eu^2 - 3/2 u.u),
// while the moments use the exact integers 36 w_a = 16, 4, 1:
//   36 drho = 16 h_0 + 4 sum_axis h + sum_diag h,  36 j = 4 sum_axis e h + sum_diag e h.
// In FP32 the inexact weights 1/9 and 1/36 would otherwise bias every collision's
// momentum by ~1e-8, which a freely decaying flow accumulates step after step.
//
// One step (Sec. 2.2, steps (2)-(6)), per node, fused:
//   pull   f_a(x) = g_a(x - e_a)                      eq. (streaming)
//   rho = rho0 + sum w_a h_a,  rho u* = sum e_a w_a h_a + F_b/2   eqs. (rho), (rho*velocity-star)
//   chi from the mask, U_O = V + omega z x (x - c) of the node's body
//   du = chi (U_O - u*) / (2 eta + chi),  F_VP = 2 rho du    eqs. (d-V), (force-density)
//   u = u* + du,  F = F_b + F_VP                       eq. (velocity-r)
//   g_a = f_a - (f+_a - f^eq+_a)/tau+ - (f-_a - f^eq-_a)/tau-
//         + (1 - 1/(2 tau+)) F+_a + (1 - 1/(2 tau-)) F-_a        eqs. (TRT-collision), (collision-modified)
// with f^eq of eq. (feq) and F_a of eq. (external-force-term), both taken at the
// corrected u and split into parts even (+) and odd (-) under a -> opposite(a).
// For a pair (a, opposite a) with eu = e_a.u and eF = e_a.F the parts are, in
// units of w_a,
//   h^eq+ = drho + rho (9/2 eu^2 - 3/2 u.u),  h^eq- = 3 rho eu = e.(36 j + 18 F)/12,
//   F+/w  = 9 eu eF - 3 u.F,                 F-/w  = 3 eF.
//
// The step is bound by HBM traffic: 9 loads, 9 stores and one mask byte per node
// against ~200 flops, so there is no matrix-core work here. What limits it is
// the bytes in flight: each thread owns V consecutive nodes of a row and moves
// every population with one aligned V-wide (16-byte) load and store. The pull
// from x -/+ 1 takes the missing end element from the neighbouring lane of the
// wavefront (a lane shuffle); the two lanes at a wavefront's ends load it
// themselves, with the domain sides resolved there. Which stores bypass the caches
// is the launch's choice (keep_tiles).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lbvp_device.h"
#include "lbvp_internal.h"
#include "lbvp_node.h"

namespace lbvp {
namespace {

// ------------------------------------------------------------ the step --

// One block updates tile t of a domain: tile_rows rows of tile_w nodes, V
// consecutive nodes per thread. part_buf: the partial buffer this step's record
// writes (the previous record is summed by leading blocks of the same launch).
// lds: the kernel's 2 FIN_LANES doubles.
// OFF32 (2-byte storage, vector pull form, a lattice under 4 GiB): the main
// loads and stores address a uniform population-row base plus a 32-bit per-lane
// byte offset, which the scalar-base addressing mode takes directly.
template <typename S, int V, int MODE, bool RECORD, bool FIELDS, bool MOVING = false, bool OFF32 = false>
__device__ __forceinline__ void step_body(const S* src, S* dst, const StepArgs<typename Arith<S>::R>& a, int t,
                                          int part_buf, double* lds, bool nt, int pose_k = 0)
{
    using R = typename Arith<S>::R;
    int s0 = 0, s1 = 0;          // this tile's (tile, body) force slots
    BodySource<R> bs;
    bs.uniform = false;
    bs.pose = nullptr;
    bs.near = 0;
    if constexpr (MOVING) {      // the poses at this step's time level (a domain with moving bodies)
        if (a.n_moving > 0) bs.pose = a.pose + (*a.pose_base + pose_k) * (int64_t)(MAX_MOVING * POSE_STRIDE);
    }
    s0 = a.tile_slot_ptr[t];
    s1 = a.tile_slot_ptr[t + 1];
    const int ty = t / a.tiles_x, tx = t - ty * a.tiles_x;
    const int tpr = a.tile_w / V;                       // threads per tile row (tile_w and V are powers of two)
    const int lr = (int)threadIdx.x >> __builtin_ctz((unsigned)tpr), lc = (int)threadIdx.x & (tpr - 1);
    const int j = min(ty * a.tile_rows + lr, a.ny - 1); // rows past ny idle (clamped for addressing)
    const int i0 = tx * a.tile_w + lc * V;
    const int lane = (int)(threadIdx.x & 63);
    const bool act = i0 < a.nx && ty * a.tile_rows + lr < a.ny;   // owns at least one real node
    const int n_own = act ? min(V, a.nx - i0) : 0;
    const int jm = (j == 0) ? a.ny - 1 : j - 1;     // rows are periodic
    const int jp = (j == a.ny - 1) ? 0 : j + 1;
    const int64_t r0 = (int64_t)j * a.pitch;   // mask and fields
    const int64_t l0 = (int64_t)j * a.lstride, lm = (int64_t)jm * a.lstride, lp = (int64_t)jp * a.lstride;
    // lattice pull source row of each direction (ey = 0 -> j, +1 -> j - 1,
    // -1 -> j + 1) and push target row (the opposite)
    const int64_t row_of[9] = {l0, l0, lm, l0, lp, lm, lm, lp, lp};
    const int row_idx[9] = {j, j, jm, j, jp, jm, jm, jp, jp};
    const int64_t row_to[9] = {l0, l0, lp, l0, lm, lp, lp, lm, lm};
    const int64_t P = a.plane;

    // Source plane of direction q: the pull and the AA local step read plane q,
    // the AA push step the neighbour's opposite slot. FP32 vectors, single
    // nodes and the AA steps take the x-shifted directions as single accesses
    // one element off alignment (columns i0 - 1 .. or i0 + 1 ..; both stay
    // inside the allocation: population 0 of row 0 is never shifted left, the
    // last population row (8 of row ny - 1) is never shifted right, and every
    // other population row is preceded and followed by another). FP64 and
    // FP16/BF16 vectors of the pull step load aligned and shift through lane
    // moves (FP64: 0.787 -> 0.783 ms and no line-straddling reads; FP32 measured
    // the same either way).
    constexpr bool kShifted = sizeof(S) == 4 || V == 1 || MODE != PULL;
    static_assert(MODE == PULL || kShifted, "the AA pattern needs dword-or-wider elements or one node per thread");
    // The lane-shuffle form (FP64 and 2-byte types, V > 1, pull) keeps the
    // loaded values in the storage type and decodes each node's nine just before
    // its collision, so that the packed loads, not 9 V decoded floats, stay live
    // across the tile.
    using LV = typename std::conditional<kShifted, R, S>::type;
    LV v[9][V];
    int body[V];
    // Threads without a node of their own (past the last column or row) load
    // column 0 of their (clamped) row instead: every access stays inside the
    // lattice, no branch or register clearing is needed, and their results are
    // never stored, summed or shuffled into an owned node.
    const int il = act ? i0 : 0;
    const int last = a.nx - 1 - i0;      // this thread's index of the domain's last column, if 0 .. V - 1
    // Everything the step reads is requested before anything is waited for: the
    // columns next to a thread's own where no lane move or shifted load has them
    // (at the domain's sides, what stands for the column outside it; left as the
    // storage type, for a conversion would wait), then the rows, then what depends
    // on the tile's slots. Asked for one after the other, each cost a memory latency:
    // BF16 2305 x 1153 22.5 -> 21.1 us per step, moving FP32 2048 x 1024 33.3 -> 30.6.
    const bool first_lane = kShifted ? i0 == 0 : (lane == 0 || lc == 0);
    const bool last_lane = (!kShifted && (lane == 63 || lc == tpr - 1)) || last < V;
    S left[3], right[3];
    if (MODE != AA_LOCAL && act && first_lane) {
        if (!kShifted && i0 > 0) {
#pragma unroll
            for (int m = 0; m < 3; ++m) left[m] = src[EXP[m] * P + row_of[EXP[m]] + (i0 - 1)];
        } else {
            side_column<MODE, false>(src, row_of, j, jm, jp, a, left);
        }
    }
    if (MODE != AA_LOCAL && act && last_lane) {
        if (!kShifted && last >= V) {
#pragma unroll
            for (int m = 0; m < 3; ++m) right[m] = src[EXM[m] * P + row_of[EXM[m]] + (i0 + V)];
        } else {
            side_column<MODE, true>(src, row_of, j, jm, jp, a, right);
        }
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        S raw[V];
        if constexpr (MODE == AA_LOCAL) {
            load_vec<S, V>(src + q * P + l0 + il, raw);
        } else {
            const int pq = (MODE == AA_PUSH) ? OPP[q] : q;
            if constexpr (OFF32) {
                static_assert(!kShifted && MODE == PULL, "the 32-bit form is the lane-shuffle pull form");
                load_vec<S, V>(at_off32(src + pq * P, (uint32_t)row_idx[q] * (uint32_t)a.lstride + (uint32_t)il),
                               raw);
            } else if constexpr (kShifted) {
                if (EXQ[q] == 1) load_vec_shifted<S, V>(src + pq * P + row_of[q] + (il - 1), raw);
                else if (EXQ[q] == -1) load_vec_shifted<S, V>(src + pq * P + row_of[q] + (il + 1), raw);
                else load_vec<S, V>(src + pq * P + row_of[q] + il, raw);
            } else {
                load_vec<S, V>(src + pq * P + row_of[q] + il, raw);
            }
        }
#pragma unroll
        for (int k = 0; k < V; ++k) v[q][k] = as_lv<LV>(raw[k]);
    }
    // the slots list every body with a node in the tile: with none, the tile's
    // mask is not read at all; with one, its row serves every solid node of the tile
    if (s1 - s0 == 1) {
        bs.uniform = true;
        bs.row = body_row(a.bodies + BODY_STRIDE * a.slot_body[s0]);
    }
    if constexpr (MOVING) {
        if (bs.pose) {   // once per tile: most tiles meet no moving body
            // only the bodies the tile's slots list can reach it during the
            // pose window (none for most tiles); of those, the ones whose
            // radius about this step's centre meets the tile
            uint32_t listed = 0;
            for (int s = s0; s < s1; ++s) listed |= 1u << (a.slot_body[s] - 1);
            if (listed) {
                const double x0 = (double)(tx * a.tile_w), y0 = (double)(ty * a.tile_rows);
                bs.near = listed & __builtin_amdgcn_readfirstlane(tile_near_bodies(
                                       a, bs.pose, x0, x0 + (double)(a.tile_w - 1), y0, y0 + (double)(a.tile_rows - 1)));
            }
        }
    }
    if (MOVING && bs.pose) {
#pragma unroll
        for (int k = 0; k < V; ++k) body[k] = (k < n_own) ? moving_body(a, bs.pose, bs.near, i0 + k, j) : 0;
    } else if (s1 > s0) {
        load_mask<V>(a.mask + r0 + il, body);
    } else {
#pragma unroll
        for (int k = 0; k < V; ++k) body[k] = 0;
    }

    // the columns next to the thread's own, put where the nodes below take them
    R from_left[3], from_right[3];
    if constexpr (!kShifted) {
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const R l = wave_shift_up1(dec(v[EXP[m]][V - 1]));
            from_left[m] = first_lane ? dec(left[m]) : l;
        }
        if (last < V - 1) {   // a row that ends inside the vector
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int k = 1; k < V; ++k) v[EXM[m]][k] = k - 1 == last ? right[m] : v[EXM[m]][k];
        }
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const R r = wave_shift_down1(dec(v[EXM[m]][0]));
            from_right[m] = last_lane ? dec(right[m]) : r;
        }
    } else if (MODE != AA_LOCAL) {
        if (first_lane) {
#pragma unroll
            for (int m = 0; m < 3; ++m) v[EXP[m]][0] = as_lv<LV>(left[m]);
        }
        if (last_lane) {
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int k = 0; k < V; ++k) v[EXM[m]][k] = k == last ? as_lv<LV>(right[m]) : v[EXM[m]][k];
        }
    }

    R fl_rho[V], fl_ux[V], fl_uy[V], fl_fx[V], fl_fy[V];
    double tile_drho = 0.0;
    S out[9][V];
    R prev[9];   // 2-byte storage: the even node's results, converted with the odd node's
#pragma unroll
    for (int k = 0; k < V; ++k) {
        R f[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) f[q] = dec(v[q][k]);
        if constexpr (!kShifted) {
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                f[EXP[m]] = (k == 0) ? from_left[m] : dec(v[EXP[m]][k > 0 ? k - 1 : 0]);
                f[EXM[m]] = (k == V - 1) ? from_right[m] : dec(v[EXM[m]][k < V - 1 ? k + 1 : 0]);
            }
        }
        const int i = i0 + k;
        NodeResult<R> n;
        if constexpr (sizeof(S) == 2) {
            n = collide_node_lowp<R, MOVING>(f, body[k], i, j, a, bs);
            if constexpr (V >= 2) {
                // two nodes' populations at a time, one packed conversion each
                if (k & 1) {
#pragma unroll
                    for (int q = 0; q < 9; ++q) enc2<S>(prev[q], f[q], &out[q][k - 1]);
                } else {
#pragma unroll
                    for (int q = 0; q < 9; ++q) prev[q] = f[q];
                }
            } else {
                // the packed conversion here too: a scalar one may be fused with
                // the collision's last multiply-add into a single rounding to the
                // storage type, which rounds some values differently from the
                // two roundings (to FP32, then to storage) of the vector forms
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    S two[2];
                    enc2<S>(f[q], R(0), two);
                    out[q][k] = two[0];
                }
            }
        } else {
            n = collide_node<R, MOVING, true, FIELDS>(f, body[k], i, j, a, bs);
#pragma unroll
            for (int q = 0; q < 9; ++q) out[q][k] = enc<S>(f[q]);
        }
        fl_rho[k] = n.rho;
        fl_ux[k] = n.ux;
        fl_uy[k] = n.uy;
        fl_fx[k] = n.fvx;
        fl_fy[k] = n.fvy;
        if constexpr (RECORD) {
            // penalization force of every node to LDS (tiles holding solid nodes
            // only), summed per body after the stores
            if (s1 > s0) {
                R* fv = dyn_lds<R>();
                fv[k * a.block + (int)threadIdx.x] = n.fvx;
                fv[(V + k) * a.block + (int)threadIdx.x] = n.fvy;
            }
        }
        if (k < n_own) tile_drho += (double)n.drho;
    }

    // ---- stores
    if constexpr (MODE == PULL || MODE == AA_LOCAL) {
        // own node: plane q (pull) or plane opp(q) (AA local)
        auto stores = [&](auto nt) {
            constexpr bool NT = decltype(nt)::value;
            if (n_own == V) {
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    if constexpr (OFF32)
                        store_vec<S, V, NT>(at_off32(dst + q * P, (uint32_t)j * (uint32_t)a.lstride + (uint32_t)i0), out[q]);
                    else
                        store_vec<S, V, NT>(dst + (MODE == PULL ? q : OPP[q]) * P + l0 + i0, out[q]);
                }
            } else if (n_own > 0) {  // ragged end of a row
#pragma unroll
                for (int k = 0; k < V; ++k)
                    if (k < n_own)
#pragma unroll
                        for (int q = 0; q < 9; ++q)
                            store_one<S, NT>(dst + (MODE == PULL ? q : OPP[q]) * P + l0 + i0 + k, out[q][k]);
            }
        };
        // in place every slot is read again soonest: plain stores at all sizes
        // (FP32 2048 x 1024 25.5 us per step against 26.4, 6144 x 2048 168 against 171)
        if constexpr (MODE == PULL) with_hint(nt, stores);
        else stores(std::false_type{});
        if constexpr (MODE == AA_LOCAL) {
            // the zero-gradient ghost columns that the next push step pulls from
            if (a.west == SIDE_OUTFLOW && act && i0 == 0)
#pragma unroll
                for (int m = 0; m < 3; ++m) static_cast<S*>(a.ghost_w)[m * (int64_t)a.ny + j] = out[EXP[m]][0];
            if (a.east == SIDE_OUTFLOW && act && i0 + n_own == a.nx)
#pragma unroll
                for (int k = 0; k < V; ++k)
                    if (k == n_own - 1)
#pragma unroll
                        for (int m = 0; m < 3; ++m)
                            static_cast<S*>(a.ghost_e)[m * (int64_t)a.ny + j] = out[EXM[m]][k];
        }
    } else {  // AA push: g_q(x) -> slot q of x + e_q
        const bool edge = (i0 == 0) || (i0 + V >= a.nx);
        if (act && !edge) {
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                if (EXQ[q] == 0) {
                    store_vec<S, V, false>(dst + q * P + row_to[q] + i0, out[q]);
                } else if constexpr (sizeof(S) >= 4) {
                    if (EXQ[q] == 1) store_vec_shifted<S, V>(dst + q * P + row_to[q] + (i0 + 1), out[q]);
                    else store_vec_shifted<S, V>(dst + q * P + row_to[q] + (i0 - 1), out[q]);
                } else {
#pragma unroll
                    for (int k = 0; k < V; ++k) store_one<S, false>(dst + q * P + row_to[q] + i0 + k + EXQ[q], out[q][k]);
                }
            }
        } else if (act) {
            // node by node, with the domain sides resolved
#pragma unroll
            for (int k = 0; k < V; ++k) {
                if (k < n_own) {
                    const int i = i0 + k;
#pragma unroll
                    for (int q = 0; q < 9; ++q) {
                        int c = i + EXQ[q];
                        bool keep = true;
                        if (c < 0) {
                            keep = (a.west == SIDE_PERIODIC);   // else it leaves the domain
                            c = a.nx - 1;
                        } else if (c >= a.nx) {
                            keep = (a.east == SIDE_PERIODIC);
                            c = 0;
                        }
                        if (keep) store_one<S, false>(dst + q * P + row_to[q] + c, out[q][k]);
                    }
                    // populations entering through a non-periodic side, for the next step
                    if (i == 0 && a.west != SIDE_PERIODIC) {
#pragma unroll
                        for (int m = 0; m < 3; ++m) {
                            const int q = EXP[m];
                            if (a.west == SIDE_INFLOW_EQ) store_one<S, false>(dst + q * P + l0, enc<S>(a.feq_in[q]));
                            else store_one<S, false>(dst + q * P + row_to[q], out[q][k]);
                        }
                    }
                    if (i == a.nx - 1 && a.east != SIDE_PERIODIC) {
#pragma unroll
                        for (int m = 0; m < 3; ++m) {
                            const int q = EXM[m];
                            if (a.east == SIDE_INFLOW_EQ) store_one<S, false>(dst + q * P + l0 + i, enc<S>(a.feq_in[q]));
                            else store_one<S, false>(dst + q * P + row_to[q] + i, out[q][k]);
                        }
                    }
                }
            }
        }
    }

    if constexpr (FIELDS) {
        R* fb = a.fields + r0 + i0;
        const int64_t F = a.plane_f;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (k < n_own) {
                fb[k] = fl_rho[k];
                fb[F + k] = fl_ux[k];
                fb[2 * F + k] = fl_uy[k];
                fb[3 * F + k] = fl_fx[k];
                fb[4 * F + k] = fl_fy[k];
            }
        }
    }

    if constexpr (RECORD) {
        // mass: one partial per wavefront (DPP moves only, no block barrier)
        double* mass_part = a.mass_part + part_buf * a.fin.mass_stride;
        double* slot_force = a.slot_force + part_buf * a.fin.slot_stride;
        const double wm = wave_sum_lane63(tile_drho);
        if (lane == 63) mass_part[(int64_t)t * (a.block >> 6) + (threadIdx.x >> 6)] = wm;
        // forces: only tiles that hold solid nodes (uniform across the block)
        // each (tile, body) slot: every wavefront sums its lanes with DPP moves
        // into lane 63, which parks the sum in LDS; after one barrier per batch
        // of slots the block's first threads add the wavefronts in order
        const R* fv = dyn_lds<R>();
        const int nw = a.block >> 6, wid = (int)threadIdx.x >> 6;
        const int per_pass = FIN_LANES / nw;          // slots whose wave sums fit lds[2 FIN_LANES]
        for (int c0 = s0; c0 < s1; c0 += per_pass) {
            const int c1 = min(s1, c0 + per_pass);
            for (int s = c0; s < c1; ++s) {
                const int b = a.slot_body[s];
                // slots of moving bodies are dense (every tile, every body): a body
                // whose radius misses this tile adds zero, without the wave sums
                // (uniform across the block)
                const bool skip = MOVING && bs.pose && !((bs.near >> (b - 1)) & 1u);
                double wx = 0.0, wy = 0.0;
                if (!skip) {
                    double px = 0.0, py = 0.0;
#pragma unroll
                    for (int k = 0; k < V; ++k) {
                        if (k < n_own && body[k] == b) {
                            px -= (double)fv[k * a.block + (int)threadIdx.x];
                            py -= (double)fv[(V + k) * a.block + (int)threadIdx.x];
                        }
                    }
                    wx = wave_sum_lane63(px);
                    wy = wave_sum_lane63(py);
                }
                if (lane == 63) {
                    lds[2 * ((s - c0) * nw + wid)] = wx;
                    lds[2 * ((s - c0) * nw + wid) + 1] = wy;
                }
            }
            __syncthreads();
            for (int s = c0 + (int)threadIdx.x; s < c1; s += a.block) {
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
}

// Two lattices: source and destination never alias.
template <typename S, int V, bool RECORD, bool FIELDS, bool MOVING = false, bool OFF32 = false>
__global__ void __launch_bounds__(256)
k_step(const S* __restrict__ src, S* __restrict__ dst, StepArgs<typename Arith<S>::R> a)
{
    __shared__ double lds[2 * FIN_LANES];   // the record sums, then the per-wavefront sums
    // the first 8 blocks sum the previous step's record (no block waits on them)
    const int lead = a.fin_n > 0 ? N_XCD : 0;
    if ((int)blockIdx.x < lead) {
        finalize_record(a.fin, a.fin_buf, a.fin_n, (int)blockIdx.x, N_XCD, lds);
        return;
    }
    const int t = xcd_tile(a.tiles_per_xcd, a.band_log2, lead);
    if (t >= a.n_tiles) return;  // whole block
    step_body<S, V, PULL, RECORD, FIELDS, MOVING, OFF32>(src, dst, a, t, a.part_buf, lds,
                                                          ((int)blockIdx.x - lead) / N_XCD >= a.keep_tiles, a.pose_k);
}

// One lattice, read and written in place (no restrict).
template <typename S, int V, int MODE, bool RECORD, bool FIELDS, bool MOVING = false>
__global__ void __launch_bounds__(256) k_step_aa(S* lat, StepArgs<typename Arith<S>::R> a)
{
    __shared__ double lds[2 * FIN_LANES];
    const int lead = a.fin_n > 0 ? N_XCD : 0;
    if ((int)blockIdx.x < lead) {
        finalize_record(a.fin, a.fin_buf, a.fin_n, (int)blockIdx.x, N_XCD, lds);
        return;
    }
    const int t = xcd_tile(a.tiles_per_xcd, a.band_log2, lead);
    if (t >= a.n_tiles) return;  // whole block
    step_body<S, V, MODE, RECORD, FIELDS, MOVING>(lat, lat, a, t, a.part_buf, lds, false, a.pose_k);
}

// Many domains in one launch: block -> (domain, tile) through the tile map;
// every domain's arguments (geometry, parameters, lattices) live in device
// memory. All domains take the same step kind, record flag and partial buffers.
template <typename S, int V, int MODE, bool RECORD, bool FIELDS, bool MOVING = false, bool OFF32 = false>
__global__ void __launch_bounds__(256) k_step_batch(BatchLaunch b)
{
    using R = typename Arith<S>::R;
    __shared__ double lds[2 * FIN_LANES];
    const StepArgs<R>* args = static_cast<const StepArgs<R>*>(b.args);
    // the first n_fin blocks sum the domains' previous records, fin_share blocks
    // per domain: dispatched first and spread over the XCDs, they overlap the
    // streaming tiles instead of trailing them (n_fin is a multiple of 8)
    if ((int)blockIdx.x < b.n_fin) {
        const int d = (int)blockIdx.x / b.fin_share;
        if (d < b.n_domains)
            finalize_record(args[d].fin, b.fin_buf, 1, (int)blockIdx.x - d * b.fin_share, b.fin_share, lds);
        return;
    }
    const int g = xcd_tile(b.tiles_per_xcd, b.band_log2, b.n_fin);
    if (g >= b.total_tiles) return;  // whole block
#if defined(__HIP_DEVICE_COMPILE__)
    // the tile map and the members' arguments do not change during a launch:
    // read through the constant address space they are scalar loads that no
    // store of the step can alias, and the arguments are copied once, up front
    // (through a generic reference every later use reloaded them)
    using CI = const __attribute__((address_space(4))) int32_t;
    using CA = const __attribute__((address_space(4))) StepArgs<R>;
    const int d = ((CI*)b.tile_domain)[g];
    const StepArgs<R> a = ((CA*)args)[d];
    const int t = g - ((CI*)b.tile_start)[d];
#else
    const int d = b.tile_domain[g];
    const StepArgs<R>& a = args[d];
    const int t = g - b.tile_start[d];
#endif
    const int cur = a.cur ^ b.flip;
    S* lat_cur = static_cast<S*>(cur ? a.lat1 : a.lat0);
    S* lat_next = static_cast<S*>(cur ? a.lat0 : a.lat1);
    step_body<S, V, MODE, RECORD, FIELDS, MOVING, OFF32>(lat_cur, MODE == PULL ? lat_next : lat_cur, a, t, b.part_buf,
                                                         lds, ((int)blockIdx.x - b.n_fin) / N_XCD >= b.keep_tiles, b.pose_k);
}

// ------------------------------------------------------------ launches --

template <typename R>
size_t record_lds_bytes(int v, int block)
{
    return 2 * (size_t)v * (size_t)block * sizeof(R);
}

template <typename S, int V, bool MOVING = false>
hipError_t step_v(int mode, bool record, bool fields, const S* in, S* out, const StepArgs<typename Arith<S>::R>& a,
                  hipStream_t s)
{
    const dim3 grid((unsigned)(a.tiles_per_xcd * N_XCD + (a.fin_n > 0 ? N_XCD : 0))), block((unsigned)a.block);
    const size_t lds = record_lds_bytes<typename Arith<S>::R>(V, a.block);
    if (mode == PULL) {
        if constexpr (sizeof(S) == 2 && V > 1) {
            if (a.off32) {
                if (record) {
                    if (fields) hipLaunchKernelGGL((k_step<S, V, true, true, MOVING, true>), grid, block, lds, s, in, out, a);
                    else hipLaunchKernelGGL((k_step<S, V, true, false, MOVING, true>), grid, block, lds, s, in, out, a);
                } else {
                    if (fields) hipLaunchKernelGGL((k_step<S, V, false, true, MOVING, true>), grid, block, 0, s, in, out, a);
                    else hipLaunchKernelGGL((k_step<S, V, false, false, MOVING, true>), grid, block, 0, s, in, out, a);
                }
                return hipGetLastError();
            }
        }
        if (record) {
            if (fields) hipLaunchKernelGGL((k_step<S, V, true, true, MOVING>), grid, block, lds, s, in, out, a);
            else hipLaunchKernelGGL((k_step<S, V, true, false, MOVING>), grid, block, lds, s, in, out, a);
        } else {
            if (fields) hipLaunchKernelGGL((k_step<S, V, false, true, MOVING>), grid, block, 0, s, in, out, a);
            else hipLaunchKernelGGL((k_step<S, V, false, false, MOVING>), grid, block, 0, s, in, out, a);
        }
        return hipGetLastError();
    }
    if constexpr (sizeof(S) >= 4 || V == 1) {
        if (mode == AA_PUSH) {
            if (record) {
                if (fields) hipLaunchKernelGGL((k_step_aa<S, V, AA_PUSH, true, true, MOVING>), grid, block, lds, s, out, a);
                else hipLaunchKernelGGL((k_step_aa<S, V, AA_PUSH, true, false, MOVING>), grid, block, lds, s, out, a);
            } else {
                if (fields) hipLaunchKernelGGL((k_step_aa<S, V, AA_PUSH, false, true, MOVING>), grid, block, 0, s, out, a);
                else hipLaunchKernelGGL((k_step_aa<S, V, AA_PUSH, false, false, MOVING>), grid, block, 0, s, out, a);
            }
        } else {
            if (record) {
                if (fields) hipLaunchKernelGGL((k_step_aa<S, V, AA_LOCAL, true, true, MOVING>), grid, block, lds, s, out, a);
                else hipLaunchKernelGGL((k_step_aa<S, V, AA_LOCAL, true, false, MOVING>), grid, block, lds, s, out, a);
            } else {
                if (fields) hipLaunchKernelGGL((k_step_aa<S, V, AA_LOCAL, false, true, MOVING>), grid, block, 0, s, out, a);
                else hipLaunchKernelGGL((k_step_aa<S, V, AA_LOCAL, false, false, MOVING>), grid, block, 0, s, out, a);
            }
        }
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;  // AA with sub-dword vectors: not built (one node per thread is)
    }
}

template <typename S>
hipError_t step_typed(int mode, bool record, bool fields, const void* src, void* dst, const void* args_v,
                      hipStream_t s)
{
    using R = typename Arith<S>::R;
    const StepArgs<R>& a = *static_cast<const StepArgs<R>*>(args_v);
    const S* in = static_cast<const S*>(src);
    S* out = static_cast<S*>(dst);
    constexpr int VW = 16 / (int)sizeof(S);
    if (a.vec == VW) return step_v<S, VW>(mode, record, fields, in, out, a, s);
    if (a.vec == 1) return step_v<S, 1>(mode, record, fields, in, out, a, s);
    if constexpr (sizeof(S) == 2) {   // 2-byte types also run 4 nodes (8 bytes) per thread
        if (a.vec == 4) return step_v<S, 4>(mode, record, fields, in, out, a, s);
    }
    return hipErrorInvalidValue;
}

template <typename S>
hipError_t step_typed_moving(int mode, bool record, bool fields, const void* src, void* dst, const void* args_v,
                             hipStream_t s)
{
    using R = typename Arith<S>::R;
    const StepArgs<R>& a = *static_cast<const StepArgs<R>*>(args_v);
    const S* in = static_cast<const S*>(src);
    S* out = static_cast<S*>(dst);
    constexpr int VW = 16 / (int)sizeof(S);
    if (a.vec == VW) return step_v<S, VW, true>(mode, record, fields, in, out, a, s);
    if (a.vec == 1) return step_v<S, 1, true>(mode, record, fields, in, out, a, s);
    if constexpr (sizeof(S) == 2) {
        if (a.vec == 4) return step_v<S, 4, true>(mode, record, fields, in, out, a, s);
    }
    return hipErrorInvalidValue;
}

template <typename S, int V, int MODE, bool MOVING>
hipError_t batch_mode(bool record, bool fields, const BatchLaunch& b, int32_t block, hipStream_t s)
{
    const dim3 grid((unsigned)(b.tiles_per_xcd * N_XCD + b.n_fin)), blk((unsigned)block);
    const size_t lds = record_lds_bytes<typename Arith<S>::R>(V, block);
    if constexpr (sizeof(S) == 2 && V > 1 && MODE == PULL) {
        if (b.off32) {
            if (record) {
                if (fields) hipLaunchKernelGGL((k_step_batch<S, V, MODE, true, true, MOVING, true>), grid, blk, lds, s, b);
                else hipLaunchKernelGGL((k_step_batch<S, V, MODE, true, false, MOVING, true>), grid, blk, lds, s, b);
            } else {
                if (fields) hipLaunchKernelGGL((k_step_batch<S, V, MODE, false, true, MOVING, true>), grid, blk, 0, s, b);
                else hipLaunchKernelGGL((k_step_batch<S, V, MODE, false, false, MOVING, true>), grid, blk, 0, s, b);
            }
            return hipGetLastError();
        }
    }
    if (record) {
        if (fields) hipLaunchKernelGGL((k_step_batch<S, V, MODE, true, true, MOVING>), grid, blk, lds, s, b);
        else hipLaunchKernelGGL((k_step_batch<S, V, MODE, true, false, MOVING>), grid, blk, lds, s, b);
    } else {
        if (fields) hipLaunchKernelGGL((k_step_batch<S, V, MODE, false, true, MOVING>), grid, blk, 0, s, b);
        else hipLaunchKernelGGL((k_step_batch<S, V, MODE, false, false, MOVING>), grid, blk, 0, s, b);
    }
    return hipGetLastError();
}

template <typename S, int V, bool MOVING>
hipError_t batch_v(int32_t mode, bool record, bool fields, const BatchLaunch& b, int32_t block, hipStream_t s)
{
    if (mode == PULL) return batch_mode<S, V, PULL, MOVING>(record, fields, b, block, s);
    if constexpr (sizeof(S) >= 4 || V == 1) {
        if (mode == AA_PUSH) return batch_mode<S, V, AA_PUSH, MOVING>(record, fields, b, block, s);
        return batch_mode<S, V, AA_LOCAL, MOVING>(record, fields, b, block, s);
    } else {
        return hipErrorInvalidValue;
    }
}

// moving: some member has moving bodies (every member then runs the kernel
// that evaluates a moving mask where a domain has one)
template <typename S, bool MOVING>
hipError_t batch_typed(int32_t vec, int32_t mode, bool record, bool fields, const BatchLaunch& b, int32_t block,
                       hipStream_t s)
{
    constexpr int VW = 16 / (int)sizeof(S);
    if (vec == VW) return batch_v<S, VW, MOVING>(mode, record, fields, b, block, s);
    if (vec == 1) return batch_v<S, 1, MOVING>(mode, record, fields, b, block, s);
    if constexpr (sizeof(S) == 2) {
        if (vec == 4) return batch_v<S, 4, MOVING>(mode, record, fields, b, block, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

template <typename S>
hipError_t StepLaunch<S>::one(bool moving, int32_t mode, bool record, bool fields, const void* src, void* dst,
                              const void* step_args, hipStream_t s)
{
    if (moving) return step_typed_moving<S>(mode, record, fields, src, dst, step_args, s);
    return step_typed<S>(mode, record, fields, src, dst, step_args, s);
}

template <typename S>
hipError_t StepLaunch<S>::batch(bool moving, int32_t vec, int32_t block, int32_t mode, bool record, bool fields,
                                const BatchLaunch& b, hipStream_t s)
{
    if (moving) return batch_typed<S, true>(vec, mode, record, fields, b, block, s);
    return batch_typed<S, false>(vec, mode, record, fields, b, block, s);
}

}  // namespace lbvp
