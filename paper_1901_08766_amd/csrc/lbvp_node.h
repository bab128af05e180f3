// lbvp_node.h -- the D2Q9 node update (moments, penalization, collision), the
// moving-mask lookup, the domain sides and the record sum, shared by the step
// kernels (lbvp_step.h) and the small kernels of lbvp_kernels.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbvp_device.h"
#include "lbvp_internal.h"

namespace lbvp {
namespace {

template <typename R>
struct NodeResult {
    R drho, rho, ux, uy, fvx, fvy;
};

// One row of the body table (see StepArgs::bodies): the centre split into its
// nearest integer and the remainder, then V and omega.
template <typename R>
struct BodyRow {
    R cxi, cyi, cxf, cyf, vx, vy, om;
};

template <typename R>
__device__ __forceinline__ BodyRow<R> body_row(const R* B)
{
    return {B[0], B[1], B[2], B[3], B[4], B[5], B[6]};
}

// Where a solid node finds its body's row: `uniform` when every solid node of
// the tile belongs to one body, whose row was then read once per tile (scalar
// loads, before any store); otherwise each node reads its own row.
template <typename R>
struct BodySource {
    bool uniform;
    BodyRow<R> row;
    const double* pose;   // moving bodies: the poses at this step's time level, else null
    uint32_t near;        // moving bodies whose reach meets the tile (bit b - 1 for body b)
};

// Volume penalization of a solid node (eqs. d-V, force-density): U_O = V +
// omega z x (x - c), du = (U_O - u*) / (2 eta + 1), F_VP = 2 rho du, u = u* + du.
// x - c comes from the split centre (a centre rounded to FP32 whole would be off
// by up to half an FP32 spacing, 1/512 node near x = 32768, the same for every
// node of the body); a moving body's centre at time t is FP64.
template <typename R, bool MOVING>
__device__ __forceinline__ void penalize(const BodySource<R>& src, int body, int i, int j, const StepArgs<R>& a,
                                         R rho, R& ux, R& uy, R& fvx, R& fvy)
{
    BodyRow<R> B;
    if (src.uniform) B = src.row;
    else B = body_row(a.bodies + BODY_STRIDE * body);
    R rx, ry;
    if (MOVING && src.pose) {
        const double* m = src.pose + (body - 1) * POSE_STRIDE;
        rx = (R)((double)i - m[2]);
        ry = (R)((double)j - m[3]);
    } else {
        rx = ((R)i - B.cxi) - B.cxf;
        ry = ((R)j - B.cyi) - B.cyf;
    }
    const R uox = B.vx - B.om * ry;
    const R uoy = B.vy + B.om * rx;
    const R dux = a.vp_c * (uox - ux);
    const R duy = a.vp_c * (uoy - uy);
    fvx = R(2) * rho * dux;
    fvy = R(2) * rho * duy;
    ux += dux;
    uy += duy;
}

// Steps (4)-(6) of the algorithm at node (i, j) with streamed populations f;
// overwrites f with the post-collision populations.
// EXACT_MOM: the odd equilibrium from the momentum (momentum3); the 2-byte
// storage types take 3 rho u as (3 rho) u instead, whose ~1e-8 momentum bias is
// far below their own rounding, for two fewer quotients per node.
// FIELDS: the node's density and velocity are stored.
template <typename R, bool MOVING = false, bool EXACT_MOM = true, bool FIELDS = false>
__device__ __forceinline__ NodeResult<R> collide_node(R (&f)[9], int body, int i, int j, const StepArgs<R>& a,
                                                    const BodySource<R>& bs)
{
    // moments with the integers 36 w_a = 16, 4, 1 (sum w_a rho0 = rho0 and
    // sum e_a w_a = 0 drop out); 1/36 and 1/rho through div36 / recip
    const R s36 = R(16) * f[0] + (R(4) * ((f[1] + f[2]) + (f[3] + f[4])) + ((f[5] + f[6]) + (f[7] + f[8])));
    const R drho = div36(s36);
    const R rho = a.rho0 + drho;
    const R d57 = f[5] - f[7], d86 = f[8] - f[6];
    const R inv_36rho = recip<FIELDS>(R(36) * rho);
    // u* = (j + F_b/2) / rho with 36 j = 4 (h1 - h3) + ... (eq. rho*velocity-star)
    const R jx36 = R(4) * (f[1] - f[3]) + (d57 + d86) + a.fbx18;
    const R jy36 = R(4) * (f[2] - f[4]) + (d57 - d86) + a.fby18;
    R ux = jx36 * inv_36rho;
    R uy = jy36 * inv_36rho;

    // volume penalization (eqs. d-V, force-density) on solid nodes only
    R fvx = R(0), fvy = R(0);
    if (body) penalize<R, MOVING>(bs, body, i, j, a, rho, ux, uy, fvx, fvy);
    const R Fx = a.fbx + fvx, Fy = a.fby + fvy;
    R px, py;   // 3 rho u
    if constexpr (EXACT_MOM) {
        px = momentum3(jx36, fvx);
        py = momentum3(jy36, fvy);
    } else {
        const R rho3 = R(3) * rho;
        px = rho3 * ux;
        py = rho3 * uy;
    }

    NodeTerms<R> n;
    const R uu = ux * ux + uy * uy;
    n.A = drho - (R(1.5) * rho) * uu;
    n.rho45 = R(4.5) * rho;
    n.uF3 = R(-3) * (ux * Fx + uy * Fy);
    const R g0 = a.om_p * (n.A - f[0]) + f[0] + a.k_p * n.uF3;
    const Pair<R> p13 = collide_pair(f[1], f[3], ux, px, Fx, n, a);
    const Pair<R> p24 = collide_pair(f[2], f[4], uy, py, Fy, n, a);
    const Pair<R> p57 = collide_pair(f[5], f[7], ux + uy, px + py, Fx + Fy, n, a);
    const Pair<R> p68 = collide_pair(f[6], f[8], uy - ux, py - px, Fy - Fx, n, a);
    f[0] = g0;
    f[1] = p13.ga;
    f[3] = p13.gb;
    f[2] = p24.ga;
    f[4] = p24.gb;
    f[5] = p57.ga;
    f[7] = p57.gb;
    f[6] = p68.ga;
    f[8] = p68.gb;
    return {drho, rho, ux, uy, fvx, fvy};
}

// The same steps for the 2-byte storage types, whose stored values carry a
// rounding error (~1e-3 relative) far above any FP32 arithmetic detail, in the
// fewest operations: 1/36 and 1/rho as single roundings, the odd equilibrium as
// (3 rho) e.u, and each pair's two relaxations regrouped into
//   g_a     = c1 h_a + c2 h_opp + (E+ + E-),
//   g_opp   = c2 h_a + c1 h_opp + (E+ - E-),
//   E+ = om_p h^eq+ + k_p F+/w = eu (9/2 om_p rho eu + 9 k_p eF) + B,
//   E- = om_m h^eq- + k_m F-/w = 3 om_m rho eu + 3 k_m eF,
//   B  = om_p (drho - 3/2 rho u.u) - 3 k_p u.F,
// with c1 = 1 - (om_p + om_m)/2, c2 = (om_m - om_p)/2 (algebraically the
// relaxation of collide_pair); the rest population is g_0 = (1 - om_p) h_0 + B.
// About 85 operations per node instead of about 125.
template <typename R, bool MOVING = false>
__device__ __forceinline__ NodeResult<R> collide_node_lowp(R (&f)[9], int body, int i, int j, const StepArgs<R>& a,
                                                         const BodySource<R>& bs)
{
    const R s36 = R(16) * f[0] + (R(4) * ((f[1] + f[2]) + (f[3] + f[4])) + ((f[5] + f[6]) + (f[7] + f[8])));
    const R drho = s36 * R(1.0 / 36.0);
    const R rho = a.rho0 + drho;
    const R d57 = f[5] - f[7], d86 = f[8] - f[6];
    const R inv_36rho = __builtin_amdgcn_rcpf(R(36) * rho);
    const R jx36 = R(4) * (f[1] - f[3]) + (d57 + d86) + a.fbx18;
    const R jy36 = R(4) * (f[2] - f[4]) + (d57 - d86) + a.fby18;
    R ux = jx36 * inv_36rho;
    R uy = jy36 * inv_36rho;
    R fvx = R(0), fvy = R(0);
    if (body) penalize<R, MOVING>(bs, body, i, j, a, rho, ux, uy, fvx, fvy);
    const R Fx = a.fbx + fvx, Fy = a.fby + fvy;
    const R uu = ux * ux + uy * uy;
    const R uF = ux * Fx + uy * Fy;
    const R B0 = a.om_p * drho - (a.om_p15 * (rho * uu) + a.k_p3 * uF);
    const R a1 = a.om_p45 * rho;
    const R r3m = a.om_m3 * rho;
    const R g0 = a.om_p1 * f[0] + B0;
    auto pair = [&](R& ha, R& hb, R eu, R eF) {
        const R t = a1 * eu + a.k_p9 * eF;
        const R ep = eu * t + B0;
        const R em = r3m * eu + a.k_m3 * eF;
        const R sum = ep + em, dif = ep - em;
        const R ga = a.c1 * ha + (a.c2 * hb + sum);
        const R gb = a.c2 * ha + (a.c1 * hb + dif);
        ha = ga;
        hb = gb;
    };
    pair(f[1], f[3], ux, Fx);
    pair(f[2], f[4], uy, Fy);
    pair(f[5], f[7], ux + uy, Fx + Fy);
    pair(f[6], f[8], uy - ux, Fy - Fx);
    f[0] = g0;
    return {drho, rho, ux, uy, fvx, fvy};
}

// Moving masks: the body occupying node (i, j) at the step's time level. Node
// x belongs to body b when the reference (t = 0) mask holds b at the node
// nearest to R(-th) (x - c(t)) + c(0), the node carried back by the body's
// rigid motion; the first such body in order wins. Evaluated in FP64 one
// operation per statement (no fused multiply-adds), so that membership does
// not depend on the storage type. Only the bodies in `near` are tried (the
// tile's, see tile_near_bodies); nodes outside a body's radius skip it.
template <typename R>
__device__ __forceinline__ int moving_body(const StepArgs<R>& a, const double* row, uint32_t near, int i, int j)
{
    for (uint32_t bits = near; bits; bits &= bits - 1) {
        const int b = __builtin_ctz(bits);
        const double* m = row + b * POSE_STRIDE;
        const double dx = (double)i - m[2];
        const double dy = (double)j - m[3];
        const double dx2 = dx * dx;
        const double dy2 = dy * dy;
        if (dx2 + dy2 > m[6]) continue;
        const double a1 = m[0] * dx;
        const double a2 = m[1] * dy;
        const double s1 = a1 + a2;
        const double xr = s1 + m[4];
        const double b1 = m[0] * dy;
        const double b2 = m[1] * dx;
        const double s2 = b1 - b2;
        const double yr = s2 + m[5];
        const double fx = floor(xr + 0.5);
        const double fy = floor(yr + 0.5);
        if (fx < 0.0 || fy < 0.0 || fx >= (double)a.nx || fy >= (double)a.ny) continue;
        if (a.mask[(int64_t)fy * a.pitch + (int64_t)fx] == b + 1) return b + 1;
    }
    return 0;
}

// The moving bodies whose radius reaches the rectangle [x0, x1] x [y0, y1] (a
// tile), as bits. Skipping the others for the tile's nodes changes nothing:
// rounding is monotone, so a node's FP64 squared distance to a centre, computed
// as in moving_body, is never below the rectangle's computed the same way.
template <typename R>
__device__ __forceinline__ uint32_t tile_near_bodies(const StepArgs<R>& a, const double* row, double x0, double x1,
                                                     double y0, double y1)
{
    uint32_t near = 0;
    for (int b = 0; b < a.n_moving; ++b) {
        const double* m = row + b * POSE_STRIDE;
        const double ex = m[2] < x0 ? x0 - m[2] : (m[2] > x1 ? m[2] - x1 : 0.0);
        const double ey = m[3] < y0 ? y0 - m[3] : (m[3] > y1 ? m[3] - y1 : 0.0);
        const double ex2 = ex * ex;
        const double ey2 = ey * ey;
        if (!(ex2 + ey2 > m[6])) near |= 1u << b;
    }
    return near;
}

// D2Q9 directions (eq. D2Q9) and the opposite map (Sec. 2.1: f_{-1} = f_3).
constexpr int OPP[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};
constexpr int EXQ[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
// Directions by x component, with rows ey = 0, +1, -1 for m = 0, 1, 2.
constexpr int EXP[3] = {1, 5, 8};   // ex = +1: pulled from column i - 1
constexpr int EXM[3] = {3, 6, 7};   // ex = -1: pulled from column i + 1

// Step kinds. PULL: two lattices, g(n) -> g(n + 1), every node pulls its nine
// populations from its neighbours' slots of the source lattice. The AA pattern
// runs on one lattice in two alternating kinds:
//   AA_PUSH  (n even) reads g_q(x - e_q) from slot opp(q) of the neighbour and
//            writes g_q(x) into slot q of the neighbour x + e_q, so that the
//            lattice then holds the streamed populations in place;
//   AA_LOCAL (n odd) reads its own slots q and writes its own slots opp(q).
// Each slot is read and written by one node only, so one buffer suffices. The
// domain sides: in AA_PUSH populations leaving through a non-periodic side are
// dropped and the ones entering are written into the boundary node's slots
// (inflow: the equilibrium; zero-gradient outflow: the boundary column's own
// outgoing value); the outflow values that AA_PUSH pulls come from a ghost
// column that AA_LOCAL writes, because the lattice slot holding them is
// overwritten by a neighbour in the same kernel.
enum Mode { PULL = 0, AA_PUSH = 1, AA_LOCAL = 2 };

// What row j's boundary column (EAST: the last) pulls from the column outside the
// domain: populations EXP of a west side, EXM of an east one. A NEIGHBOR side (a
// cut of a slab decomposition) reads the halo column that lbvp_halo_exchange wrote
// into the current lattice's padding (column nx for the east side, pitch - 1 for
// the west; a context with a cut has pitch >= nx + 2), so it is one more column
// choice, like a periodic side. Ghost populations are values of the storage type,
// like every other population (the AA push step stores the inflow ones in the
// lattice), so the inflow equilibrium is rounded to it.
template <int MODE, bool EAST, typename S, typename R>
__device__ __forceinline__ void side_column(const S* src, const int64_t (&row_of)[9], int j, int jm, int jp,
                                            const StepArgs<R>& a, S (&e)[3])
{
    const int side = EAST ? a.east : a.west;
    if (side == SIDE_INFLOW_EQ) {
#pragma unroll
        for (int m = 0; m < 3; ++m) e[m] = enc<S>(a.feq_in[EAST ? EXM[m] : EXP[m]]);
    } else if (MODE == AA_PUSH && side == SIDE_OUTFLOW) {
        const S* ghost = static_cast<const S*>(EAST ? a.ghost_e : a.ghost_w);
        const int rows[3] = {j, jm, jp};
#pragma unroll
        for (int m = 0; m < 3; ++m) e[m] = ghost[m * (int64_t)a.ny + rows[m]];
    } else {
        const int c = EAST ? (side == SIDE_PERIODIC ? 0 : (side == SIDE_NEIGHBOR ? a.nx : a.nx - 1))
                           : (side == SIDE_PERIODIC ? a.nx - 1 : (side == SIDE_NEIGHBOR ? (int)a.pitch - 1 : 0));
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int q = EAST ? EXM[m] : EXP[m], pq = MODE == AA_PUSH ? OPP[q] : q;
            e[m] = src[pq * a.plane + row_of[q] + c];
        }
    }
}

// ------------------------------------------------------------ the record --

// The FIN_LANES virtual lanes' values in sx and sy (LDS) summed pairwise with
// halving spans (128, 64, ... 1); thread 0 gets the two sums. The first two
// levels are additions of values that lane l of the first wavefront reads itself,
// the other six lane moves, so that a sum costs one barrier, not one per level.
__device__ __forceinline__ void record_tree(const double* sx, const double* sy, double* x, double* y)
{
    __syncthreads();
    if (threadIdx.x < 64) {
        const int l = (int)threadIdx.x;
        double u = (sx[l] + sx[l + 128]) + (sx[l + 64] + sx[l + 192]);
        double v = (sy[l] + sy[l + 128]) + (sy[l + 64] + sy[l + 192]);
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) {
            u += __shfl_down(u, w, 64);
            v += __shfl_down(v, w, 64);
        }
        *x = u;
        *y = v;
    }
    __syncthreads();   // sx and sy are reused by the next sum
}

// Share blk of n_blk blocks (n_blk divides FIN_COUNTERS) of the sums of n_rec
// records, in partial buffers buf, buf + 1, ... : a record's mass and every one
// of its bodies are a unit each, dealt out in turn, so that the sums
// of a record, each a chain of dependent loads and a tree, run side by side.
// With one block doing them one after the other, the chain outlasted the step of
// a small domain: 64 x 64 nodes in FP64 with two bodies took 10.9 us a step.
// Every sum has an order fixed by the data alone: the partials are dealt to
// FIN_LANES virtual lanes (lane_sum, or slot by slot), which meet in
// record_tree; neither the block size nor n_blk changes a record by one bit.
// Each share counts the records itself: counters blk, blk + n_blk, ... are its
// own, so no block waits for another.
__device__ __forceinline__ void finalize_record(const FinalizeArgs& f, int buf, int n_rec, int blk, int n_blk, double* lds)
{
    double* sx = lds;
    double* sy = lds + FIN_LANES;
    const int64_t count = f.rec_count[blk];
    const int per = f.n_bodies + 1;
    for (int unit = blk; unit < n_rec * per; unit += n_blk) {
        const int rec = unit / per, b = unit - rec * per - 1;   // b = -1: the mass
        const int64_t pb = (buf + rec) & (f.n_buf - 1), r = (count + rec) % f.capacity;
        const double* pm = f.mass_part + pb * f.mass_stride;
        const double* sf = f.slot_force + pb * f.slot_stride;
        if (b < 0) {
            for (int v = (int)threadIdx.x; v < FIN_LANES; v += (int)blockDim.x) {
                sx[v] = lane_sum(pm, f.n_mass, v);
                sy[v] = 0.0;
            }
        } else {
            const int s0 = f.body_slot_ptr[b], s1 = f.body_slot_ptr[b + 1];
            for (int v = (int)threadIdx.x; v < FIN_LANES; v += (int)blockDim.x) {
                double x = 0.0, y = 0.0;
                int k = s0 + v;
                // four slots' loads in flight at a time, added in the same order
                for (; k + 3 * FIN_LANES < s1; k += 4 * FIN_LANES) {
                    int sl[4];
                    double px[4], py[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) sl[u] = f.body_slots[k + u * FIN_LANES];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        px[u] = sf[2 * sl[u]];
                        py[u] = sf[2 * sl[u] + 1];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        x += px[u];
                        y += py[u];
                    }
                }
                for (; k < s1; k += FIN_LANES) {
                    const int sl = f.body_slots[k];
                    x += sf[2 * sl];
                    y += sf[2 * sl + 1];
                }
                sx[v] = x;
                sy[v] = y;
            }
        }
        double x = 0.0, y = 0.0;
        record_tree(sx, sy, &x, &y);
        if (threadIdx.x == 0) {
            if (b < 0) {
                f.ring_mass[r] = f.mass_offset + x;
            } else {
                f.ring_force[(r * f.max_bodies + b) * 2] = x;
                f.ring_force[(r * f.max_bodies + b) * 2 + 1] = y;
            }
        }
    }
    if (threadIdx.x == 0)
        for (int c = blk; c < FIN_COUNTERS; c += n_blk) f.rec_count[c] = count + n_rec;
}

}  // namespace
}  // namespace lbvp
