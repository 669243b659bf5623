// lbm_kernels.hip -- gfx950 kernels of the plane-strain LBM
// (Schlueter et al., arXiv 2301.00228).
//
// One time step is one launch of k_interior:
//
//  k_interior  every body node of every plate, tiled.  A workgroup owns a
//              strip of columns and marches up a band of rows.  Each lane
//              loads its node's populations once, collides them (eq. LBE,
//              dt/tau = 2) and hands the post-collision populations and the
//              zeroth moments to its x-neighbours through LDS and to its
//              y-neighbours through registers.  Interior nodes then take the
//              acceleration of eq. navier from the neighbours' phi and psi,
//              advance u and du/dt by eq. integration, and (unless a
//              neighbour is a boundary node) store the streamed populations.
//              Workgroups whose tile or halo ring holds boundary or
//              second-row nodes first finish the previous step there (the
//              prologue): the boundary reset of eqs. psi_phi_at_bound and
//              correction-f, the second-row pull of eq. LBE_mod with the
//              time-averaged boundary populations, and the boundary
//              accelerations of eqs. acc_neumann / acc_dirichlet with their
//              Newmark update.  The latency of that work hides behind the
//              other workgroups' streaming.
//  k_boundary  the same boundary work for every boundary node, one block
//              per chunk of boundary nodes; it closes each run of steps (and
//              precedes every synchronization) so the state is complete.
//  k_sync      the synchronization of Sec. 3.2 every l steps.
//
// Populations, u and du/dt ping-pong through two buffers (a third holds the
// intermediate time level of two-step launches).  The march never writes
// boundary or second-row nodes: boundary nodes keep their populations of
// t_{n-1} in the previous buffer, which the prologue reads, and second-row
// nodes' pulls go to a small side buffer (two of them, by step parity) that
// the next step's boundary work completes.  Boundary nodes' u(t_{n+1}) is
// written one step ahead.
#include <hip/hip_runtime.h>

#include <mutex>

#include "../../include/lbm.h"
#include "lbm_device.h"
#include "lbm_kernels.h"
#include "lbm_types.h"

namespace lbm {

// ------------------------------------------- boundary / second-row work

// Flux of eq. correction-f under reading R2 at boundary node (i, j) with
// class byte cl, field fl: the first moment (lattice units) of the
// post-collision populations (eq. LBE, dt/tau = 2) that the LBE would
// stream into the node at t from its body neighbours x - c^alpha, their
// populations at t - dt being in buffer po (those neighbours are boundary
// or second-row nodes, whose populations the march never overwrites); a
// missing neighbour contributes 0.
template <class CD>
__device__ void streamed_in_flux(const DevState &s, const PlateDev &P, int i, int j, uint8_t cl,
                                 int fl, int po, typename CD::C &jx, typename CD::C &jy) {
  using C = typename CD::C;
  using Slot = typename CD::Slot;
  // population alpha arrives from x - c^alpha: 1 from W, 2 from S, 3 from E,
  // 4 from N (one neighbour at a time)
  C sx = C(0), sy = C(0);
#pragma unroll 1
  for (int al = 1; al < 5; al++) {
    const int di = (al == 1) - (al == 3), dj = (al == 2) - (al == 4);
    const uint8_t from = al == 1 ? NB_W : al == 2 ? NB_S : al == 3 ? NB_E : NB_N;
    if (!(cl & from)) continue;
    const int64_t ky = node_of(P, wrapc(i - di, P.nx), wrapc(j - dj, P.ny));
    Slot r[5];
    CD::load_raw(s, po, fl, ky, r);
    C rho, fs[5];
    CD::collide_raw(P, fl, r, rho, fs);
    // fs[al] (a select, not a dynamic index into a local array)
    const C g = al == 1 ? fs[1] : al == 2 ? fs[2] : al == 3 ? fs[3] : fs[4];
    if (di != 0) sx += C(di) * g;
    if (dj != 0) sy += C(dj) * g;
  }
  jx = sx;
  jy = sy;
}

// Inputs of one boundary task read from memory: the flux of eq.
// correction-f of both fields and u, du/dt at t.
template <class CD>
struct BoundaryIn {
  typename CD::C jx[2], jy[2];
  typename CD::U ux, uy, vx, vy;
};

// The reads of one boundary task (see boundary_task): the flux from the
// populations at t - dt in buffer po (reading R1, or R2 for variant
// contexts) if reset, u and du/dt from buffer ua if accel.  Kept apart from
// the arithmetic so that a caller can issue them early.
template <class CD, bool VAR>
__device__ __forceinline__ void boundary_load(const DevState &s, const PlateDev &P, const BTask &T,
                                              int po, bool reset, bool accel, int ua,
                                              BoundaryIn<CD> &in) {
  using U = typename CD::U;
  const BndNode &B = T.b;
  const int64_t k = B.node;
  if (reset) {
    if (VAR && (P.readings & RD_FLUX_STREAMED)) {
      const uint8_t cl = s.cls[k];
      streamed_in_flux<CD>(s, P, B.i, B.j, cl, 0, po, in.jx[0], in.jy[0]);
      streamed_in_flux<CD>(s, P, B.i, B.j, cl, 1, po, in.jx[1], in.jy[1]);
    } else {
      CD::flux(s, po, 0, k, P, in.jx[0], in.jy[0]);
      CD::flux(s, po, 1, k, P, in.jx[1], in.jy[1]);
    }
  }
  if (accel) {
    in.ux = ldg<U>(s.u[ua][0], k);
    in.uy = ldg<U>(s.u[ua][1], k);
    in.vx = ldg<U>(s.v[ua][0], k);
    in.vy = ldg<U>(s.v[ua][1], k);
  }
}

// One boundary node.  grad: rows of 4 gradient values (d_x u_x, d_y u_x,
// d_x u_y, d_y u_y) of u at time t, indexed by the task's g[].
//  reset (eqs. psi_phi_at_bound, correction-f): populations at t from the
//    field div u / (curl u).e_z and the flux in `in`, written to buffer pn;
//  accel (eq. acc_dirichlet or eq. acc_neumann, step n with loads at n dt /
//    (n+1) dt): from u, du/dt at t in `in`, Newmark update (eq.
//    integration) into buffer ub (and ub2 if >= 0).
template <class CD>
__device__ __forceinline__ void boundary_finish(const DevState &s, const PlateDev &P, const BTask &T,
                                const typename CD::U *grad, const BoundaryIn<CD> &in, int pn,
                                bool reset, bool accel, int ub, int ub2, unsigned long long n) {
  using C = typename CD::C;
  using U = typename CD::U;
  const BndNode &B = T.b;
  const int64_t k = B.node;
  const U *gs = grad + 4 * T.g[0];
  if (reset) {
    const U dv = gs[0] + gs[3];
    const U cu = gs[2] - gs[1];
    CD::store_eq(s, pn, 0, k, P, (C)dv, in.jx[0], in.jy[0]);
    CD::store_eq(s, pn, 1, k, P, (C)cu, in.jx[1], in.jy[1]);
  }
  if (!accel) return;
  const U ux0 = in.ux, uy0 = in.uy, vx0 = in.vx, vy0 = in.vy;
  U ax, ay;
  if (B.kind == LBM_BC_DIRICHLET) {
    const double g = load_amp(s, B.load, (double)(n + 1) * P.dt);
    dirichlet_accel<U>(P, n, (U)(g * B.val[0]), (U)(g * B.val[1]), ux0, uy0, vx0, vy0, ax, ay);
  } else {
    const double g = load_amp(s, B.load, (double)n * P.dt);
    const U l[4] = {(U)B.cell[1], (U)B.cell[2], (U)B.cell[3], (U)B.cell[4]};
    U sk[3], sr[4][3];
    bool has[4];
    hooke<U>(P, gs, sk[0], sk[1], sk[2]);
#pragma unroll
    for (int d = 0; d < 4; d++) {
      has[d] = T.g[1 + d] >= 0;
      sr[d][0] = sr[d][1] = sr[d][2] = U(0);
      if (has[d]) hooke<U>(P, grad + 4 * T.g[1 + d], sr[d][0], sr[d][1], sr[d][2]);
    }
    neumann_accel<U>(P, sk, has, sr, (U)B.cell[0], l, (U)(g * B.val[0]), (U)(g * B.val[1]), ax, ay);
  }
  U nux, nuy, nvx, nvy;
  newmark<U>(P, kick_of<U>(P, n == 0), ax, ay, ux0, uy0, vx0, vy0, nux, nuy, nvx, nvy);
  stg<U>(s.u[ub][0], k, nux);
  stg<U>(s.u[ub][1], k, nuy);
  stg<U>(s.v[ub][0], k, nvx);
  stg<U>(s.v[ub][1], k, nvy);
  if (ub2 >= 0) {
    stg<U>(s.u[ub2][0], k, nux);
    stg<U>(s.u[ub2][1], k, nuy);
    stg<U>(s.v[ub2][0], k, nvx);
    stg<U>(s.v[ub2][1], k, nvy);
  }
  if (!(fabs((double)nux) < 1e30) || !(fabs((double)nuy) < 1e30)) s.flag[0] = 1;
}

// One boundary node's reset and acceleration (reads from buffers po and ua,
// writes to pn, ub, ub2; see boundary_load and boundary_finish).
template <class CD, bool VAR>
__device__ void boundary_task(const DevState &s, const PlateDev &P, const BTask &T,
                              const typename CD::U *grad, int po, int pn, bool reset, bool accel,
                              int ua, int ub, int ub2, unsigned long long n) {
  BoundaryIn<CD> in;
  boundary_load<CD, VAR>(s, P, T, po, reset, accel, ua, in);
  boundary_finish<CD>(s, P, T, grad, in, pn, reset, accel, ub, ub2, n);
}

// Population AL that second-row node Q pulls from its upwind boundary node
// y = x - c^AL by eq. LBE_mod under the plate's readings (used when they are
// not R1 + M1): the average of y's populations at t - dt (buffer po) and of
// their reset values at t (field from grad, flux of eq. correction-f by
// reading R1 or R2), collided towards the equilibrium of its own moments (M1)
// or of y's populations at t - dt (M2).
template <class CD, int AL>
__device__ typename CD::C pull_from_boundary(const DevState &s, const PlateDev &P, const STask &Q,
                                             int fl, const typename CD::U *grad, int po) {
  using C = typename CD::C;
  using U = typename CD::U;
  using Slot = typename CD::Slot;
  constexpr int di = (AL == 1) - (AL == 3), dj = (AL == 2) - (AL == 4);
  const int yi = wrapc(Q.i - di, P.nx), yj = wrapc(Q.j - dj, P.ny);
  const int64_t ky = node_of(P, yi, yj);
  Slot raw[5];
  CD::load_raw(s, po, fl, ky, raw);
  const U *gy = grad + 4 * Q.g[AL];
  const C fld = fl == 0 ? (C)(gy[0] + gy[3]) : (C)(gy[2] - gy[1]);
  C jx, jy, f[5], fnew[5];
  if (P.readings & RD_FLUX_STREAMED)
    streamed_in_flux<CD>(s, P, yi, yj, s.cls[ky], fl, po, jx, jy);
  else
    CD::raw_flux(raw, jx, jy);
  CD::eq_pops(P, fl, fld, jx, jy, fnew);
  CD::raw_to_pops(P, fl, raw, f);
#pragma unroll
  for (int q = 0; q < 5; q++) f[q] = C(0.5) * (fnew[q] + f[q]);
  if (P.readings & RD_EQ_OLD) {
    // f~ - 2 (f~ - f_eq(rho, J of the populations at t - dt))
    C jox, joy, e[5];
    CD::raw_flux(raw, jox, joy);
    CD::eq_pops(P, fl, CD::raw_rho(raw), jox, joy, e);
    return f[AL] - C(2.0) * (f[AL] - e[AL]);
  }
  C r, fs[5];
  collide_pops<CD>(P, fl, f, r, fs);
  return fs[AL];
}

// Inputs of one field of one second-row task read from memory (readings
// R1 and M1): the side buffer's pulls and the stored state at t - dt of its
// first upwind boundary node (direction a1, 0 if none).
template <class CD>
struct SecondRowIn {
  typename CD::C fo[5];
  typename CD::Slot raw[5];
  int a1;
};

template <class CD>
__device__ __forceinline__ void second_row_load(const DevState &s, const PlateDev &P,
                                                const STask &Q, int fl, int po, int sr,
                                                SecondRowIn<CD> &in) {
  using C = typename CD::C;
  const C *side = static_cast<const C *>(s.side[sr]);
#pragma unroll
  for (int al = 0; al < 5; al++) in.fo[al] = side[(int64_t)(fl * 5 + al) * s.nsec + Q.si];
  in.a1 = Q.g[1] >= 0 ? 1 : Q.g[2] >= 0 ? 2 : Q.g[3] >= 0 ? 3 : Q.g[4] >= 0 ? 4 : 0;
  if (in.a1 != 0) {
    const int di = (in.a1 == 1) - (in.a1 == 3), dj = (in.a1 == 2) - (in.a1 == 4);
    const int64_t ky = node_of(P, wrapc(Q.i - di, P.nx), wrapc(Q.j - dj, P.ny));
    CD::load_raw(s, po, fl, ky, in.raw);
  }
}

// One field of one second-row node: its populations at t, pulled from the
// upwind nodes at t - dt.  Those pulled from non-boundary upwind nodes were
// left in the side buffer by the march of the previous step (in.fo); one
// leaving a boundary node follows eq. LBE_mod: the average of the boundary
// node's populations at t - dt (buffer po; in.raw for the first such node)
// and of their reset values at t (field from grad, flux of eq. correction-f
// by reading R1: that of the populations at t - dt), collided with the
// equilibrium of their own moments (reading M1).  Written to buffer pn.
template <class CD>
__device__ __forceinline__ void second_row_finish(const DevState &s, const PlateDev &P, const STask &Q, int fl,
                                  const typename CD::U *grad, int po, int pn,
                                  const SecondRowIn<CD> &in) {
  using C = typename CD::C;
  using U = typename CD::U;
  using Slot = typename CD::Slot;
  C fo[5];
#pragma unroll
  for (int al = 0; al < 5; al++) fo[al] = in.fo[al];
#pragma unroll
  for (int al = 1; al < 5; al++) {
    if (Q.g[al] < 0) continue;
    Slot raw[5];
    if (al == in.a1) {
#pragma unroll
      for (int q = 0; q < 5; q++) raw[q] = in.raw[q];
    } else {
      // a further upwind boundary node (a corner)
      const int di = (al == 1) - (al == 3), dj = (al == 2) - (al == 4);
      const int64_t ky = node_of(P, wrapc(Q.i - di, P.nx), wrapc(Q.j - dj, P.ny));
      CD::load_raw(s, po, fl, ky, raw);
    }
    C f[5], r, fs[5];
    CD::raw_to_pops(P, fl, raw, f);
    const U *gy = grad + 4 * Q.g[al];
    const C fld = fl == 0 ? (C)(gy[0] + gy[3]) : (C)(gy[2] - gy[1]);
    C fnew[5], jx, jy;
    CD::raw_flux(raw, jx, jy);
    CD::eq_pops(P, fl, fld, jx, jy, fnew);
#pragma unroll
    for (int qq = 0; qq < 5; qq++) f[qq] = C(0.5) * (fnew[qq] + f[qq]);
    collide_pops<CD>(P, fl, f, r, fs);
    fo[al] = fs[al];
  }
  CD::store(s, pn, fl, Q.node, P, fo);
}

// One field of one second-row node under the plate's readings (buffers po,
// pn, side buffer sr): R1 and M1 by second_row_load and second_row_finish;
// the variant readings (VAR contexts only) through pull_from_boundary.
template <class CD, bool VAR>
__device__ void second_row_task(const DevState &s, const PlateDev &P, const STask &Q, int fl,
                                const typename CD::U *grad, int po, int pn, int sr) {
  using C = typename CD::C;
  if (VAR && P.readings != 0) {
    const C *side = static_cast<const C *>(s.side[sr]);
    C fo[5];
#pragma unroll
    for (int al = 0; al < 5; al++) fo[al] = side[(int64_t)(fl * 5 + al) * s.nsec + Q.si];
    if (Q.g[1] >= 0) fo[1] = pull_from_boundary<CD, 1>(s, P, Q, fl, grad, po);
    if (Q.g[2] >= 0) fo[2] = pull_from_boundary<CD, 2>(s, P, Q, fl, grad, po);
    if (Q.g[3] >= 0) fo[3] = pull_from_boundary<CD, 3>(s, P, Q, fl, grad, po);
    if (Q.g[4] >= 0) fo[4] = pull_from_boundary<CD, 4>(s, P, Q, fl, grad, po);
    CD::store(s, pn, fl, Q.node, P, fo);
    return;
  }
  SecondRowIn<CD> in;
  second_row_load<CD>(s, P, Q, fl, po, sr, in);
  second_row_finish<CD>(s, P, Q, fl, grad, po, pn, in);
}

// Prologue of an interior tile at step n (buffers sb): the boundary work
// (readings R1 and M1 only: contexts with other readings run every step's
// boundary work in k_boundary) of step n - 1 for the boundary and
// second-row nodes of the tile and its
// halo ring (resets and pulls into buffer sb.in, which the march then reads,
// from the populations of t_{n-1} in buffer sb.prev and the side buffer
// sb.sp) and the next boundary accelerations of the tile's own boundary
// nodes (u buffer sb.in to sb.out).  Gradients of u(t_n) go to LDS (lds,
// lds_bytes: the march's exchange buffer, unused until the march starts) if
// they fit, else to a per-tile scratch area in global memory.  `plate` is
// the tile's plate (the chunk's).
//
// The prologue is a chain of dependent memory reads on a tile's critical
// path.  Each lane's first gradient node, boundary task and second-row task
// therefore read their records first and then all their inputs (stencil
// values of u, the flux and u, du/dt of the boundary node, the side-buffer
// pulls and the first upwind boundary node's state) before any of them is
// used, so that the chain is records -> inputs -> barrier -> arithmetic and
// stores; further items (lists longer than the workgroup) follow one by one.
template <class CD>
__device__ void prologue(const DevState &s, const Prologue &pro, int chunk, int plate,
                         const StepBufs &sb, int tid, int nthreads, void *lds, int lds_bytes) {
  using U = typename CD::U;
  const TileChunk ch = pro.chunks[chunk];
  const PlateDev P = s.plates[plate];
  const bool in_lds = (int64_t)(ch.g1 - ch.g0) * 4 * (int64_t)sizeof(U) <= (int64_t)lds_bytes;
  U *grad = in_lds ? static_cast<U *>(lds) : static_cast<U *>(pro.grad) + (int64_t)4 * ch.g0;
  const U *ux = static_cast<const U *>(s.u[sb.in][0]);
  const U *uy = static_cast<const U *>(s.u[sb.in][1]);
  const unsigned long long n = s.counter[sb.in];
  const int nst = 2 * (ch.s1 - ch.s0);
  const int g = ch.g0 + tid, b = ch.b0 + tid;
  const bool hg = g < ch.g1, hb = b < ch.b1, hs = tid < nst;
  TGradNode G{};
  BTask T{};
  STask Q{};
  if (hg) G = pro.gn[g];
  if (hb) T = pro.bt[b];
  if (hs) Q = pro.st[ch.s0 + (tid >> 1)];
  U gu[2][5];
  if (hg) {
    const int cx = G.code & 7, cy = (G.code >> 3) & 7;
    fd_stencil_values<U>(ux, P, G.i, G.j, cx, cy, gu[0]);
    fd_stencil_values<U>(uy, P, G.i, G.j, cx, cy, gu[1]);
  }
  BoundaryIn<CD> bin;
  if (hb) boundary_load<CD, false>(s, P, T, sb.prev, true, T.accel != 0, sb.in, bin);
  SecondRowIn<CD> sin;
  if (hs) second_row_load<CD>(s, P, Q, tid & 1, sb.prev, sb.sp, sin);
  for (int g2 = g; g2 < ch.g1; g2 += nthreads) {
    if (g2 != g) {
      G = pro.gn[g2];
      const int cx = G.code & 7, cy = (G.code >> 3) & 7;
      fd_stencil_values<U>(ux, P, G.i, G.j, cx, cy, gu[0]);
      fd_stencil_values<U>(uy, P, G.i, G.j, cx, cy, gu[1]);
    }
    const int cx = G.code & 7, cy = (G.code >> 3) & 7;
    U *d = grad + 4 * (g2 - ch.g0);
    d[0] = fd_vals<U>(cx, gu[0][0], gu[0][1], gu[0][2], P);
    d[1] = fd_vals<U>(cy, gu[0][0], gu[0][3], gu[0][4], P);
    d[2] = fd_vals<U>(cx, gu[1][0], gu[1][1], gu[1][2], P);
    d[3] = fd_vals<U>(cy, gu[1][0], gu[1][3], gu[1][4], P);
  }
  __syncthreads();
  for (int b2 = b; b2 < ch.b1; b2 += nthreads) {
    if (b2 != b) {
      T = pro.bt[b2];
      boundary_load<CD, false>(s, P, T, sb.prev, true, T.accel != 0, sb.in, bin);
    }
    boundary_finish<CD>(s, P, T, grad, bin, sb.in, true, T.accel != 0, sb.out, -1, n);
  }
  for (int t = tid; t < nst; t += nthreads) {
    if (t != tid) {
      Q = pro.st[ch.s0 + (t >> 1)];
      second_row_load<CD>(s, P, Q, t & 1, sb.prev, sb.sp, sin);
    }
    second_row_finish<CD>(s, P, Q, t & 1, grad, sb.prev, sb.in, sin);
  }
  __syncthreads();
}

// Boundary work of step n - 1 for every boundary node, one block per chunk
// of boundary nodes (all of one plate): the same work as the prologues of
// step n.  The state of t_n is in buffer bc, the boundary populations of
// t_{n-1} in bp, the second-row pulls in side[sr].  Phase 1 puts u(t_n) of
// every node the chunk's stencils touch into LDS, phase 2 the
// finite-difference gradients; phase 3 runs the boundary tasks (reset into
// buffer bc if do_reset; acceleration into u buffer ub, and ub2 if >= 0) and,
// if do_reset, the second-row tasks (one field per thread).
template <int ST>
__global__ void __launch_bounds__(kBoundaryThreads)
    k_boundary(DevState s, const Chunk *__restrict__ chunks, const UNode *__restrict__ un,
               const GradNode *__restrict__ gn, const BTask *__restrict__ btask,
               const STask *__restrict__ stask, int bc, int bp, int ub, int ub2, int sr,
               int do_reset) {
  using CD = typename CodecOf<ST>::type;
  using U = typename CD::U;
  __shared__ U uu[kMaxU][2];
  __shared__ U grad[kMaxGrad][4];
  const Chunk ch = chunks[blockIdx.x];
  const PlateDev P = s.plates[ch.plate];
  const int tid = threadIdx.x;
  for (int g = ch.u0 + tid; g < ch.u1; g += kBoundaryThreads) {
    const int64_t k = un[g].node;
    uu[g - ch.u0][0] = ldg<U>(s.u[bc][0], k);
    uu[g - ch.u0][1] = ldg<U>(s.u[bc][1], k);
  }
  __syncthreads();
  for (int g = ch.g0 + tid; g < ch.g1; g += kBoundaryThreads) {
    const GradNode G = gn[g];
    const int cx = G.code & 7, cy = (G.code >> 3) & 7;
    U *d = grad[g - ch.g0];
#pragma unroll
    for (int c = 0; c < 2; c++) {
      const U q0 = uu[G.u[0]][c];
      d[2 * c + 0] = fd_vals<U>(cx, q0, uu[G.u[1]][c], uu[G.u[2]][c], P);
      d[2 * c + 1] = fd_vals<U>(cy, q0, uu[G.u[3]][c], uu[G.u[4]][c], P);
    }
  }
  __syncthreads();
  const unsigned long long n = s.counter[bc];
  const int nb = ch.b1 - ch.b0;
  if (tid < nb) {
    const BTask T = btask[ch.b0 + tid];
    boundary_task<CD, true>(s, P, T, &grad[0][0], bp, bc, do_reset != 0, true, bc, ub, ub2, n);
  } else if (do_reset) {
    const int t = tid - nb;
    if (ch.s0 + (t >> 1) < ch.s1)
      second_row_task<CD, true>(s, P, stask[ch.s0 + (t >> 1)], t & 1, &grad[0][0], bp, bc, sr);
  }
}

// -------------------------------------------------------- interior kernel

// Exchange slots in LDS per lane and row.
enum { X_RHO0 = 0, X_RHO1, X_F1_0, X_F1_1, X_F3_0, X_F3_1, X_N };

// LDS rows of the x-exchange per march stage.  Each row is published one
// iteration before it is read, with one barrier per iteration.  Several
// waves need three rows (a wave one barrier ahead may publish the next row
// while another still reads the previous one); a single wave executes its
// LDS accesses in order, so two rows suffice, which leaves LDS room for
// more waves per CU.
__host__ __device__ constexpr int ex_rows(int lanes) { return lanes == 64 ? 2 : 3; }

// Two steps of a tile whose area and two-node halo ring hold only interior
// nodes (no boundary or second-row node): step n on the area plus its
// one-node ring (from t_n on the two-node ring, buffer sb.in), step n + 1 on
// the area (buffer sb.out2); the t_{n+1} populations of the export bands
// (owned columns / rows next to single-step tiles) go to buffer sb.out.  Lane
// l holds column x0 - 2 + l.  Rows are indexed i = 0..h-1 in the march
// direction (i = -2, -1, h, h+1: halo rows).  The front row a of t_n is
// collided while row a - 1 takes step n and row a - 2 step n + 1; each
// stage hands its post-collision values to the x-neighbours through its own
// triple-buffered LDS slots (exA: t_n, exB: t_{n+1}).  deep: a launch of
// deep tiles, never the run's first step (it does not read the step
// counters, which the launches beside it may be writing).
template <class CD, int TWL, bool NT>
__device__ void march2(const DevState &s, const Tile &t, const StepBufs &sb,
                       typename CD::C (*exA)[X_N][TWL], typename CD::C (*exB)[X_N][TWL],
                       bool deep) {
  using C = typename CD::C;
  using U = typename CD::U;
  using Slot = typename CD::Slot;
  const PlateDev P = s.plates[t.plate];
  const int lane = threadIdx.x;
  const int w = t.x1 - t.x0;
  const bool live = lane <= w + 3;
  const int x = wrapc(t.x0 - 2 + lane, P.nx);
  const bool stepA = lane >= 1 && lane <= w + 2;  // step n on columns x0-1 .. x1
  const bool stepB = lane >= 2 && lane <= w + 1;  // step n+1 on the owned columns
  const int d = t.dir ? -1 : 1;
  const int h = t.y1 - t.y0;
  auto row_y = [&](int i) { return wrapc(d > 0 ? t.y0 + i : t.y1 - 1 - i, P.ny); };
  // Every lane loads (lanes past the tile from column x0, their values are
  // not used): a load under a branch, or a default written over the
  // registers of a load in flight, makes the compiler wait for all
  // outstanding memory operations right there.
  const int xl = live ? x : t.x0;
  auto load_raw = [&](int i, Slot raw[2][5]) {
    const int64_t k = node_of(P, xl, row_y(i));
    CD::load_raw(s, sb.in, 0, k, raw[0]);
    CD::load_raw(s, sb.in, 1, k, raw[1]);
  };
  auto load_uv = [&](int i, U uv[4]) {
    const int64_t k = node_of(P, xl, row_y(i));
    uv[0] = ldg<U>(s.u[sb.in][0], k);
    uv[1] = ldg<U>(s.u[sb.in][1], k);
    uv[2] = ldg<U>(s.v[sb.in][0], k);
    uv[3] = ldg<U>(s.v[sb.in][1], k);
  };
  auto collide_raw = [&](const Slot raw[2][5], C rho[2], C fs[2][5]) {
#pragma unroll
    for (int fl = 0; fl < 2; fl++) CD::collide_raw(P, fl, raw[fl], rho[fl], fs[fl]);
  };
  // t_n values of lanes past the tile (their loads read column x0)
  auto clear_dead = [&](C rho[2], C fs[2][5]) {
    if (!live) {
#pragma unroll
      for (int fl = 0; fl < 2; fl++) {
        rho[fl] = C(0);
#pragma unroll
        for (int qq = 0; qq < 5; qq++) fs[fl][qq] = C(0);
      }
    }
  };
  auto publish = [&](C(*ex)[X_N][TWL], int slot, const C rho[2], const C fs[2][5]) {
    ex[slot][X_RHO0][lane] = rho[0];
    ex[slot][X_RHO1][lane] = rho[1];
    ex[slot][X_F1_0][lane] = fs[0][1];
    ex[slot][X_F1_1][lane] = fs[1][1];
    ex[slot][X_F3_0][lane] = fs[0][3];
    ex[slot][X_F3_1][lane] = fs[1][3];
  };
  // population a row streams into the row after it (behind) / before it
  auto behind_pop = [&](const C fs[5]) { return d > 0 ? fs[2] : fs[4]; };
  auto ahead_pop = [&](const C fs[5]) { return d > 0 ? fs[4] : fs[2]; };
  constexpr int NS = ex_rows(TWL);
  auto slot_of = [](int i) { return (i + 3 * NS) % NS; };  // i >= -3
  // Pull into row i of one stage: f0 of the row, f1 / f3 from the x
  // neighbours (slot of row i), the behind row's and the ahead row's pops;
  // then the u, du/dt update from the neighbours' rho.
  auto finalize = [&](C(*ex)[X_N][TWL], int i, const C f0[2], const C fbe[2], const C fah[2],
                      const C rbe[2], const C rah[2], const U uv[4], C f[2][5], U nu[4],
                      const Kick<U> &K) {
    const int sl = slot_of(i);
    // (the end lanes read a clamped neighbour; their results are not used)
    const int lw = lane > 0 ? lane - 1 : 0, le = lane < TWL - 1 ? lane + 1 : TWL - 1;
#pragma unroll
    for (int fl = 0; fl < 2; fl++) {
      f[fl][0] = f0[fl];
      f[fl][1] = ex[sl][fl == 0 ? X_F1_0 : X_F1_1][lw];
      f[fl][3] = ex[sl][fl == 0 ? X_F3_0 : X_F3_1][le];
      f[fl][2] = d > 0 ? fbe[fl] : fah[fl];
      f[fl][4] = d > 0 ? fah[fl] : fbe[fl];
    }
    const C wr0 = ex[sl][X_RHO0][lw], er0 = ex[sl][X_RHO0][le];
    const C wr1 = ex[sl][X_RHO1][lw], er1 = ex[sl][X_RHO1][le];
    const C n0 = d > 0 ? rah[0] : rbe[0], s0 = d > 0 ? rbe[0] : rah[0];
    const C n1 = d > 0 ? rah[1] : rbe[1], s1 = d > 0 ? rbe[1] : rah[1];
    interior_update<U>(P, K, (U)er0, (U)wr0, (U)n0, (U)s0, (U)er1, (U)wr1, (U)n1, (U)s1, uv[0],
                       uv[1], uv[2], uv[3], nu[0], nu[1], nu[2], nu[3]);
  };
  // displacement-update coefficients of steps n (the run's first if n = 0)
  // and n + 1
  const Kick<U> kickA = kick_of<U>(P, !deep && s.counter[sb.in] == 0ull),
                kickB = kick_of<U>(P, false);

  // t_n stage registers: row a-2 (rho, behind pop), row a-1 (rho, f0, behind pop)
  C a2_rho[2], a2_fb[2], a1_rho[2], a1_f0[2], a1_fb[2];
  // t_{n+1} stage registers: row a-3 (rho, behind pop), row a-2 (rho, f0, behind pop)
  C b3_rho[2], b3_fb[2], b2_rho[2], b2_f0[2], b2_fb[2];
  U uvA[4];   // u, du/dt of t_n, row a-1 (row a once step n of row a-1 is done)
  U uvB[4];   // u, du/dt of t_{n+1}, row a-2
  Slot rawn[2][5];  // t_n populations of row a
  {
    Slot raw[2][5];
    C rho[2], fs[2][5];
    load_raw(-2, raw);
    load_raw(-1, rawn);
    collide_raw(raw, rho, fs);
    clear_dead(rho, fs);
    a2_rho[0] = rho[0];
    a2_rho[1] = rho[1];
    a2_fb[0] = behind_pop(fs[0]);
    a2_fb[1] = behind_pop(fs[1]);
#pragma unroll
    for (int fl = 0; fl < 2; fl++)
#pragma unroll
      for (int qq = 0; qq < 5; qq++) raw[fl][qq] = rawn[fl][qq];
    load_raw(0, rawn);
    load_uv(-1, uvA);
    collide_raw(raw, rho, fs);
    clear_dead(rho, fs);
    publish(exA, slot_of(-1), rho, fs);
    a1_rho[0] = rho[0];
    a1_rho[1] = rho[1];
    a1_f0[0] = fs[0][0];
    a1_f0[1] = fs[1][0];
    a1_fb[0] = behind_pop(fs[0]);
    a1_fb[1] = behind_pop(fs[1]);
#pragma unroll
    for (int q = 0; q < 4; q++) uvB[q] = U(0);
#pragma unroll
    for (int fl = 0; fl < 2; fl++)
      b3_rho[fl] = b3_fb[fl] = b2_rho[fl] = b2_f0[fl] = b2_fb[fl] = C(0);
  }
  for (int a = 0; a <= h + 1; a++) {
    // collide t_n row a and prefetch row a+1 into the registers it used
    // (the last iteration reloads row h+1)
    Slot raw[2][5];
    C rho[2], fs[2][5];
#pragma unroll
    for (int fl = 0; fl < 2; fl++)
#pragma unroll
      for (int qq = 0; qq < 5; qq++) raw[fl][qq] = rawn[fl][qq];
    load_raw(a + 1 <= h + 1 ? a + 1 : h + 1, rawn);
    collide_raw(raw, rho, fs);
    clear_dead(rho, fs);
    publish(exA, slot_of(a), rho, fs);
    __syncthreads();
    // step n at row a-1 (columns x0-1 .. x1)
    const C fa[2] = {ahead_pop(fs[0]), ahead_pop(fs[1])};
    C g[2][5];
    U nu[4];
    finalize(exA, a - 1, a1_f0, a2_fb, fa, a2_rho, rho, uvA, g, nu, kickA);
    // u of row a (for the next row's step n) into the registers just used
    load_uv(a <= h ? a : h, uvA);
    const int ya = row_y(a - 1);
    if (stepA && a - 1 >= 0 && a - 1 < h) {
      const bool exp = ((t.flags & TF_EXP_W) && lane == 2) ||
                       ((t.flags & TF_EXP_E) && lane == w + 1) ||
                       ((t.flags & TF_EXP_S) && ya == t.y0) ||
                       ((t.flags & TF_EXP_N) && ya == t.y1 - 1);
      if (exp && stepB) {
        const int64_t k = node_of(P, x, ya);
        CD::store(s, sb.out, 0, k, P, g[0]);
        CD::store(s, sb.out, 1, k, P, g[1]);
      }
    }
    // collide t_{n+1} row a-1 (as a store and a load between two launches
    // would leave it) and hand it to the x-neighbours
    C rho1[2], fs1[2][5];
    CD::collide_stored(P, 0, g[0], rho1[0], fs1[0]);
    CD::collide_stored(P, 1, g[1], rho1[1], fs1[1]);
    if (!stepA) {
#pragma unroll
      for (int fl = 0; fl < 2; fl++) {
        rho1[fl] = C(0);
#pragma unroll
        for (int qq = 0; qq < 5; qq++) fs1[fl][qq] = C(0);
      }
    }
    publish(exB, slot_of(a - 1), rho1, fs1);
    // step n+1 at row a-2 (owned columns); its x-neighbours' values were
    // published in the previous iteration
    if (a - 2 >= 0 && a - 2 < h) {
      const C fa1[2] = {ahead_pop(fs1[0]), ahead_pop(fs1[1])};
      C g2[2][5];
      U nu2[4];
      finalize(exB, a - 2, b2_f0, b3_fb, fa1, b3_rho, rho1, uvB, g2, nu2, kickB);
      if (stepB) {
        // NT: the pass's final state is not read again in this launch;
        // nontemporal stores leave the caches to the halo rows
        const int64_t k = node_of(P, x, row_y(a - 2));
        stg<U, NT>(s.u[sb.out2][0], k, nu2[0]);
        stg<U, NT>(s.u[sb.out2][1], k, nu2[1]);
        stg<U, NT>(s.v[sb.out2][0], k, nu2[2]);
        stg<U, NT>(s.v[sb.out2][1], k, nu2[3]);
        CD::template store<NT>(s, sb.out2, 0, k, P, g2[0]);
        CD::template store<NT>(s, sb.out2, 1, k, P, g2[1]);
      }
    }
    // shift the stages by one row
#pragma unroll
    for (int fl = 0; fl < 2; fl++) {
      a2_rho[fl] = a1_rho[fl];
      a2_fb[fl] = a1_fb[fl];
      a1_rho[fl] = rho[fl];
      a1_f0[fl] = fs[fl][0];
      a1_fb[fl] = behind_pop(fs[fl]);
      b3_rho[fl] = b2_rho[fl];
      b3_fb[fl] = b2_fb[fl];
      b2_rho[fl] = rho1[fl];
      b2_f0[fl] = fs1[fl][0];
      b2_fb[fl] = behind_pop(fs1[fl]);
    }
#pragma unroll
    for (int q = 0; q < 4; q++) uvB[q] = nu[q];
  }
}

// (FP64 with two-step tiles of one wave: at most 168 VGPRs, so that three
// waves fit per SIMD; with more lanes per tile LDS allows only two.)
// DEEP: a launch of deep two-step tiles (no boundary or single-step tile
// within two nodes), which runs beside the launches that own the step
// counters and so leaves them alone.
template <int ST, int TWL, bool TWO, bool DEEP, bool NT>
__global__ void __launch_bounds__(TWL)
    __attribute__((amdgpu_waves_per_eu((TWO && ST == LBM_STORE_F64 && TWL == 64) ? 3 : 1)))
    k_interior(DevState s, const Tile *__restrict__ tiles, int ntiles, int q, StepBufs sb,
               Prologue pro) {
  using CD = typename CodecOf<ST>::type;
  using C = typename CD::C;
  using U = typename CD::U;
  using Slot = typename CD::Slot;
  constexpr int NS = ex_rows(TWL);
  __shared__ __align__(16) C exs[TWO ? 2 * NS : NS][X_N][TWL];
  C(*ex)[X_N][TWL] = exs;

  // populations and u, du/dt of t_n in buffers sb.in, of t_{n+1} in sb.out
  const int pc = sb.in, pn = sb.out, uc = sb.in, un = sb.out;
  // With overlapped pairs this launch's chain (single-step and frame tiles)
  // paces the step while the deep launch runs beside it: its waves get the
  // higher instruction-issue priority on a SIMD (-1 % per step on the
  // 1024^2 plate; no effect on one stream).
  if constexpr (!DEEP) __builtin_amdgcn_s_setprio(1);
  if (!DEEP && blockIdx.x == 0 && threadIdx.x == 0) s.counter[un] = s.counter[uc] + 1ull;
  const int tix = tile_index(blockIdx.x, q);
  if (tix >= ntiles) return;
  const Tile t = tiles[tix];
  if constexpr (DEEP) {
    march2<CD, TWL, NT>(s, t, sb, exs, exs + NS, true);
    return;
  }
  if (TWO && sb.out2 >= 0 && (t.flags & TF_TWO)) {
    march2<CD, TWL, NT>(s, t, sb, exs, exs + NS, false);
    return;
  }
  if (pro.enabled && t.chunk >= 0)
    prologue<CD>(s, pro, t.chunk, t.plate, sb, (int)threadIdx.x, TWL, exs, (int)sizeof(exs));
  const PlateDev P = s.plates[t.plate];
  const Kick<U> kick = kick_of<U>(P, s.counter[sb.in] == 0ull);
  const int lane = threadIdx.x;
  // this lane's column segment: lanes 0 .. w+1 the first (a halo column on
  // each side), the next wb+2 lanes the second of a paired tile; a lane
  // reads its x-neighbours' values from lanes lane -+ 1, which for an owned
  // column are its own segment's
  const int wa = t.x1 - t.x0, wb = t.bx1 > t.bx0 ? t.bx1 - t.bx0 : 0;
  const bool segb = wb > 0 && lane >= wa + 2;
  const int sl = segb ? lane - (wa + 2) : lane;  // lane within the segment
  const int w = segb ? wb : wa;
  int x = (segb ? t.bx0 : t.x0) - 1 + sl;
  bool xok = sl <= w + 1;
  if (x < 0 || x >= P.nx) {
    if (P.periodic & 1)
      x = wrapc(x, P.nx);
    else
      xok = false;
  }
  const bool owned = xok && sl >= 1 && sl <= w;
  const bool py = (P.periodic & 2) != 0;

  // Node of row y in this lane's column; false if there is none.
  auto row_node = [&](int y, int64_t &k) -> bool {
    bool ok = xok;
    if (y < 0 || y >= P.ny) {
      if (py)
        y = wrapc(y, P.ny);
      else
        ok = false;
    }
    k = node_of(P, x, y);
    return ok;
  };
  auto load_cls = [&](int y) -> uint8_t {
    int64_t k;
    return row_node(y, k) ? s.cls[k] : (uint8_t)0;
  };
  // Raw populations of row y (only for body nodes: cl from load_cls).
  auto load_raw = [&](int y, uint8_t cl, Slot raw[2][5]) {
    int64_t k;
    const bool ok = row_node(y, k) && (cl & CL_IN);
#pragma unroll
    for (int fl = 0; fl < 2; fl++)
#pragma unroll
      for (int qq = 0; qq < 5; qq++) raw[fl][qq] = Slot(0);
    if (ok) {
      CD::load_raw(s, pc, 0, k, raw[0]);
      CD::load_raw(s, pc, 1, k, raw[1]);
    }
  };
  auto load_uv = [&](int y, uint8_t cl, U uv[4]) {
    uv[0] = uv[1] = uv[2] = uv[3] = U(0);
    if (owned && (cl & (CL_IN | CL_B)) == CL_IN) {
      const int64_t k = node_of(P, x, y);
      uv[0] = ldg<U>(s.u[uc][0], k);
      uv[1] = ldg<U>(s.u[uc][1], k);
      uv[2] = ldg<U>(s.v[uc][0], k);
      uv[3] = ldg<U>(s.v[uc][1], k);
    }
  };
  auto collide_row = [&](uint8_t cl, const Slot raw[2][5], C rho[2], C fs[2][5]) {
#pragma unroll
    for (int fl = 0; fl < 2; fl++) {
      CD::collide_raw(P, fl, raw[fl], rho[fl], fs[fl]);
      if (!(cl & CL_IN)) {
        rho[fl] = C(0);
#pragma unroll
        for (int qq = 0; qq < 5; qq++) fs[fl][qq] = C(0);
      }
    }
  };
  auto publish = [&](int slot, const C rho[2], const C fs[2][5]) {
    ex[slot][X_RHO0][lane] = rho[0];
    ex[slot][X_RHO1][lane] = rho[1];
    ex[slot][X_F1_0][lane] = fs[0][1];
    ex[slot][X_F1_1][lane] = fs[1][1];
    ex[slot][X_F3_0][lane] = fs[0][3];
    ex[slot][X_F3_1][lane] = fs[1][3];
  };

  // The march visits the rows upwards (d = +1) or downwards (d = -1, tiles
  // with dir set): vertically adjacent tiles march in opposite directions,
  // so the halo rows they share are read by both at about the same time and
  // the second read hits in L2.  "Behind" is row r - d, "ahead" row r + d.
  // Software pipeline over rows: while row r is finalized, the populations
  // of row r + 2d, u and du/dt of row r + d and the class bytes of row r + 3d
  // are in flight.
  const int d = t.dir ? -1 : 1;
  const int h = t.y1 - t.y0;
  const int r0 = t.dir ? t.y1 - 1 : t.y0;
  // rows of the tile plus its halo rows: y0 - 1 .. y1
  auto in_reach = [&](int k) { return k <= h; };  // row r0 + k d, k >= -1
  C be_rho[2], be_f[2];                  // row r - d: rho, population streaming into r
  C cu_rho[2], cu_f0[2], cu_fb[2];       // row r (cu_fb: streams into r + d)
  uint8_t cu_cl, cl1, cl2, cl3;          // classes of rows r, r + d, r + 2d, r + 3d
  Slot raw1[2][5];                       // populations of row r + d
  U uv0[4];                              // u, du/dt of row r
  // the behind row streams population 2 (d = +1, from the south) or 4 into
  // row r, the ahead row the other one
  auto behind_pop = [&](const C fs[5]) { return d > 0 ? fs[2] : fs[4]; };
  {
    const uint8_t clm = load_cls(r0 - d);
    cu_cl = load_cls(r0);
    cl1 = load_cls(r0 + d);
    cl2 = load_cls(r0 + 2 * d);
    Slot raw[2][5];
    C rho[2], fs[2][5];
    load_raw(r0 - d, clm, raw);
    collide_row(clm, raw, rho, fs);
    be_rho[0] = rho[0];
    be_rho[1] = rho[1];
    be_f[0] = behind_pop(fs[0]);
    be_f[1] = behind_pop(fs[1]);
    load_raw(r0, cu_cl, raw);
    load_raw(r0 + d, cl1, raw1);
    load_uv(r0, cu_cl, uv0);
    collide_row(cu_cl, raw, rho, fs);
    publish(0, rho, fs);
    cu_rho[0] = rho[0];
    cu_rho[1] = rho[1];
    cu_f0[0] = fs[0][0];
    cu_f0[1] = fs[1][0];
    cu_fb[0] = behind_pop(fs[0]);
    cu_fb[1] = behind_pop(fs[1]);
  }
  int slot = 0;
  for (int k = 0; k < h; k++) {
    const int r = r0 + k * d;
    const int nslot = slot + 1 == NS ? 0 : slot + 1;
    // prefetch
    cl3 = in_reach(k + 3) ? load_cls(r + 3 * d) : (uint8_t)0;
    Slot raw2[2][5];
    if (in_reach(k + 2)) {
      load_raw(r + 2 * d, cl2, raw2);
    } else {
#pragma unroll
      for (int fl = 0; fl < 2; fl++)
#pragma unroll
        for (int qq = 0; qq < 5; qq++) raw2[fl][qq] = Slot(0);
    }
    U uv1[4];
    load_uv(r + d, (k + 1 < h) ? cl1 : (uint8_t)0, uv1);
    // collide row r + d and hand its values to the x-neighbours
    C nx_rho[2], nx_fs[2][5];
    collide_row(cl1, raw1, nx_rho, nx_fs);
    publish(nslot, nx_rho, nx_fs);
    __syncthreads();
    const bool fin = owned && (cu_cl & (CL_IN | CL_B)) == CL_IN;
    if (fin) {
      const int64_t kn = node_of(P, x, r);
      const C wr0 = ex[slot][X_RHO0][lane - 1], er0 = ex[slot][X_RHO0][lane + 1];
      const C wr1 = ex[slot][X_RHO1][lane - 1], er1 = ex[slot][X_RHO1][lane + 1];
      // rho of the north / south neighbours
      const C n0 = d > 0 ? nx_rho[0] : be_rho[0], s0 = d > 0 ? be_rho[0] : nx_rho[0];
      const C n1 = d > 0 ? nx_rho[1] : be_rho[1], s1 = d > 0 ? be_rho[1] : nx_rho[1];
      U nux, nuy, nvx, nvy;
      interior_update<U>(P, kick, (U)er0, (U)wr0, (U)n0, (U)s0, (U)er1, (U)wr1, (U)n1, (U)s1,
                         uv0[0], uv0[1], uv0[2], uv0[3], nux, nuy, nvx, nvy);
      stg<U>(s.u[un][0], kn, nux);
      stg<U>(s.u[un][1], kn, nuy);
      stg<U>(s.v[un][0], kn, nvx);
      stg<U>(s.v[un][1], kn, nvy);
      // Pull: f_alpha(x, t+dt) = f*_alpha(x - c^alpha dt).  A second-row
      // node keeps it in the side buffer; the next step's boundary work
      // replaces the populations that leave boundary nodes and stores it.
      const bool sec = (cu_cl & CL_S) != 0;
      const int64_t si = sec ? (int64_t)s.sidx[kn] : 0;
      C *side = static_cast<C *>(s.side[sb.sp ^ 1]);
#pragma unroll
      for (int fl = 0; fl < 2; fl++) {
        C f[5];
        f[0] = cu_f0[fl];
        f[1] = ex[slot][fl == 0 ? X_F1_0 : X_F1_1][lane - 1];
        f[3] = ex[slot][fl == 0 ? X_F3_0 : X_F3_1][lane + 1];
        f[2] = d > 0 ? be_f[fl] : nx_fs[fl][2];
        f[4] = d > 0 ? nx_fs[fl][4] : be_f[fl];
        if (!sec) {
          CD::store(s, pn, fl, kn, P, f);
        } else {
#pragma unroll
          for (int qq = 0; qq < 5; qq++) side[(int64_t)(fl * 5 + qq) * s.nsec + si] = f[qq];
        }
      }
    }
    be_rho[0] = cu_rho[0];
    be_rho[1] = cu_rho[1];
    be_f[0] = cu_fb[0];
    be_f[1] = cu_fb[1];
    cu_rho[0] = nx_rho[0];
    cu_rho[1] = nx_rho[1];
    cu_f0[0] = nx_fs[0][0];
    cu_f0[1] = nx_fs[1][0];
    cu_fb[0] = behind_pop(nx_fs[0]);
    cu_fb[1] = behind_pop(nx_fs[1]);
    cu_cl = cl1;
    cl1 = cl2;
    cl2 = cl3;
#pragma unroll
    for (int fl = 0; fl < 2; fl++)
#pragma unroll
      for (int qq = 0; qq < 5; qq++) raw1[fl][qq] = raw2[fl][qq];
#pragma unroll
    for (int qq = 0; qq < 4; qq++) uv0[qq] = uv1[qq];
    slot = nslot;
  }
}

// Periodic synchronization (Sec. 3.2): at every body node the fields become
// the finite differences of u, the populations f_eq(field, current J).
template <int ST, int TWL>
__global__ void __launch_bounds__(TWL)
    k_sync(DevState s, const Tile *__restrict__ tiles, int ntiles, int q, int b) {
  using CD = typename CodecOf<ST>::type;
  using C = typename CD::C;
  using U = typename CD::U;
  const int tix = tile_index(blockIdx.x, q);
  if (tix >= ntiles) return;
  const Tile t = tiles[tix];
  const PlateDev P = s.plates[t.plate];
  // owned columns of the tile's first segment, then of its second
  const int wa = t.x1 - t.x0, lane = (int)threadIdx.x;
  const int x = lane < wa ? t.x0 + lane : t.bx0 + (lane - wa);
  if (lane >= wa && x >= t.bx1) return;
  for (int y = t.y0; y < t.y1; y++) {
    const int64_t k = node_of(P, x, y);
    if (!(s.cls[k] & CL_IN)) continue;
    U dv, cu;
    div_curl<U>(s, b, P, x, y, dv, cu);
    C jx, jy;
    CD::flux(s, b, 0, k, P, jx, jy);
    CD::store_eq(s, b, 0, k, P, (C)dv, jx, jy);
    CD::flux(s, b, 1, k, P, jx, jy);
    CD::store_eq(s, b, 1, k, P, (C)cu, jx, jy);
    const double ux = (double)ldg<U>(s.u[b][0], k), uy = (double)ldg<U>(s.u[b][1], k);
    if (!(fabs(ux) < 1e30) || !(fabs(uy) < 1e30)) s.flag[0] = 1;
  }
}

// Initial state of one plate (Fig. 4): u, du/dt from the dense host arrays;
// populations f_eq(field, J = 0) with the field from finite differences of
// u0 unless given directly.
template <int ST>
__global__ void k_init_uv(DevState s, int plate, const double *__restrict__ u0,
                          const double *__restrict__ v0) {
  using U = typename CodecOf<ST>::type::U;
  const PlateDev P = s.plates[plate];
  const int64_t n = (int64_t)P.nx * P.ny;
  for (int64_t d = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; d < n;
       d += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(d % P.nx), j = (int)(d / P.nx);
    const int64_t k = node_of(P, i, j);
    const bool in = (s.cls[k] & CL_IN) != 0;
    const U ux = in && u0 ? (U)u0[d] : U(0), uy = in && u0 ? (U)u0[n + d] : U(0);
    const U vx = in && v0 ? (U)v0[d] : U(0), vy = in && v0 ? (U)v0[n + d] : U(0);
    for (int b = 0; b < 2; b++) {
      stg<U>(s.u[b][0], k, ux);
      stg<U>(s.u[b][1], k, uy);
      stg<U>(s.v[b][0], k, vx);
      stg<U>(s.v[b][1], k, vy);
    }
  }
}

template <int ST>
__global__ void k_init_pops(DevState s, int plate, const double *__restrict__ e0,
                            const double *__restrict__ w0) {
  using CD = typename CodecOf<ST>::type;
  using C = typename CD::C;
  using U = typename CD::U;
  const PlateDev P = s.plates[plate];
  const int64_t n = (int64_t)P.nx * P.ny;
  for (int64_t d = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; d < n;
       d += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(d % P.nx), j = (int)(d / P.nx);
    const int64_t k = node_of(P, i, j);
    if (!(s.cls[k] & CL_IN)) continue;
    U dv, cu;
    div_curl<U>(s, 0, P, i, j, dv, cu);
    const C phi = e0 ? (C)e0[d] : (C)dv;
    const C psi = w0 ? (C)w0[d] : (C)cu;
    CD::store_eq(s, 0, 0, k, P, phi, C(0), C(0));
    CD::store_eq(s, 0, 1, k, P, psi, C(0), C(0));
  }
}

// Fields of one plate into dense FP64 device arrays (zero outside the body).
template <int ST>
__global__ void k_fields(DevState s, int plate, int b, double *e, double *w, double *u,
                         double *v) {
  using CD = typename CodecOf<ST>::type;
  using U = typename CD::U;
  const PlateDev P = s.plates[plate];
  const int64_t n = (int64_t)P.nx * P.ny;
  for (int64_t d = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; d < n;
       d += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(d % P.nx), j = (int)(d / P.nx);
    const int64_t k = node_of(P, i, j);
    const bool in = (s.cls[k] & CL_IN) != 0;
    if (e) e[d] = in ? CD::field(s, b, 0, k, P) : 0.0;
    if (w) w[d] = in ? CD::field(s, b, 1, k, P) : 0.0;
    if (u) {
      u[d] = in ? (double)ldg<U>(s.u[b][0], k) : 0.0;
      u[n + d] = in ? (double)ldg<U>(s.u[b][1], k) : 0.0;
    }
    if (v) {
      v[d] = in ? (double)ldg<U>(s.v[b][0], k) : 0.0;
      v[n + d] = in ? (double)ldg<U>(s.v[b][1], k) : 0.0;
    }
  }
}

// Consistency error of Sec. 4 (tension example): per body node the 2-norm
// of (omega - (curl u).e_z, e - div u), the fields being the sums of the
// populations and the derivatives of u the finite differences the method
// uses at that node; 0 outside the body.
template <int ST>
__global__ void k_cons_err(DevState s, int plate, int b, double *err) {
  using CD = typename CodecOf<ST>::type;
  using U = typename CD::U;
  const PlateDev P = s.plates[plate];
  const int64_t n = (int64_t)P.nx * P.ny;
  for (int64_t d = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; d < n;
       d += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(d % P.nx), j = (int)(d / P.nx);
    const int64_t k = node_of(P, i, j);
    if (!(s.cls[k] & CL_IN)) {
      err[d] = 0.0;
      continue;
    }
    U dv, cu;
    div_curl<U>(s, b, P, i, j, dv, cu);
    const double d1 = CD::field(s, b, 1, k, P) - (double)cu;
    const double d0 = CD::field(s, b, 0, k, P) - (double)dv;
    err[d] = sqrt(d1 * d1 + d0 * d0);
  }
}

// --------------------------------------------------------------- launchers

template <int ST, bool TWO, bool DEEP, bool NT>
static hipError_t launch_interior_t(const DevState &s, const Tile *tiles, int ntiles, int lanes,
                                    const StepBufs &b, const Prologue &pro, hipStream_t st) {
  // at least one block: block 0 advances the step counter
  const int q = ntiles > 0 ? (ntiles + 7) / 8 : 1;
  const dim3 grid(8 * q);
  switch (lanes) {
    case 64:
      hipLaunchKernelGGL((k_interior<ST, 64, TWO, DEEP, NT>), grid, dim3(64), 0, st, s, tiles, ntiles,
                         q, b, pro);
      break;
    case 128:
      hipLaunchKernelGGL((k_interior<ST, 128, TWO, DEEP, NT>), grid, dim3(128), 0, st, s, tiles,
                         ntiles, q, b, pro);
      break;
    case 256:
      hipLaunchKernelGGL((k_interior<ST, 256, TWO, DEEP, NT>), grid, dim3(256), 0, st, s, tiles,
                         ntiles, q, b, pro);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int ST>
static hipError_t launch_sync_t(const DevState &s, const Tile *tiles, int ntiles, int lanes,
                                int b, hipStream_t st) {
  const int q = (ntiles + 7) / 8;
  const dim3 grid(8 * q);
  switch (lanes) {
    case 64:
      hipLaunchKernelGGL((k_sync<ST, 64>), grid, dim3(64), 0, st, s, tiles, ntiles, q, b);
      break;
    case 128:
      hipLaunchKernelGGL((k_sync<ST, 128>), grid, dim3(128), 0, st, s, tiles, ntiles, q, b);
      break;
    case 256:
      hipLaunchKernelGGL((k_sync<ST, 256>), grid, dim3(256), 0, st, s, tiles, ntiles, q, b);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

#define LBM_DISPATCH(st, CALL)                                   \
  switch (st) {                                                  \
    case LBM_STORE_F64: { constexpr int ST = LBM_STORE_F64; CALL; } break;       \
    case LBM_STORE_F32: { constexpr int ST = LBM_STORE_F32; CALL; } break;       \
    case LBM_STORE_F32DEV: { constexpr int ST = LBM_STORE_F32DEV; CALL; } break; \
    case LBM_STORE_F16DEV: { constexpr int ST = LBM_STORE_F16DEV; CALL; } break; \
    case LBM_STORE_BF16DEV: { constexpr int ST = LBM_STORE_BF16DEV; CALL; } break; \
    default: return hipErrorInvalidValue;                        \
  }

hipError_t launch_interior(int st, const DevState &s, const Tile *tiles, int ntiles, int lanes,
                           const StepBufs &b, const Prologue &pro, hipStream_t stream) {
  if (b.out2 >= 0 && b.nt) {
    LBM_DISPATCH(st, return (launch_interior_t<ST, true, false, true>(s, tiles, ntiles, lanes, b,
                                                                      pro, stream)));
  } else if (b.out2 >= 0) {
    LBM_DISPATCH(st, return (launch_interior_t<ST, true, false, false>(s, tiles, ntiles, lanes, b,
                                                                       pro, stream)));
  } else {
    LBM_DISPATCH(st, return (launch_interior_t<ST, false, false, false>(s, tiles, ntiles, lanes, b,
                                                                        pro, stream)));
  }
  return hipSuccess;
}

hipError_t launch_deep(int st, const DevState &s, const Tile *tiles, int ntiles, int lanes,
                       const StepBufs &b, hipStream_t stream) {
  if (ntiles <= 0) return hipSuccess;
  if (b.out2 < 0) return hipErrorInvalidValue;
  const Prologue none{};
  if (b.nt) {
    LBM_DISPATCH(st, return (launch_interior_t<ST, true, true, true>(s, tiles, ntiles, lanes, b,
                                                                     none, stream)));
  } else {
    LBM_DISPATCH(st, return (launch_interior_t<ST, true, true, false>(s, tiles, ntiles, lanes, b,
                                                                      none, stream)));
  }
  return hipSuccess;
}

hipError_t launch_boundary(int st, const DevState &s, const Chunk *chunks, int nchunks,
                           const UNode *un, const GradNode *gn, const BTask *bt, const STask *stk,
                           int bc, int bp, int ub, int ub2, int sr, int do_reset,
                           hipStream_t stream) {
  if (nchunks <= 0) return hipSuccess;
  LBM_DISPATCH(st, hipLaunchKernelGGL((k_boundary<ST>), dim3(nchunks), dim3(kBoundaryThreads), 0,
                                      stream, s, chunks, un, gn, bt, stk, bc, bp, ub, ub2, sr,
                                      do_reset));
  return hipGetLastError();
}

hipError_t launch_sync(int st, const DevState &s, const Tile *tiles, int ntiles, int lanes, int b,
                       hipStream_t stream) {
  if (ntiles <= 0) return hipSuccess;
  LBM_DISPATCH(st, return launch_sync_t<ST>(s, tiles, ntiles, lanes, b, stream));
  return hipSuccess;
}

hipError_t launch_init(int st, const DevState &s, int plate, int64_t nodes, const double *u0,
                       const double *v0, const double *e0, const double *w0, hipStream_t stream) {
  int64_t blocks = (nodes + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  LBM_DISPATCH(st, hipLaunchKernelGGL((k_init_uv<ST>), dim3((unsigned)blocks), dim3(256), 0,
                                      stream, s, plate, u0, v0));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  LBM_DISPATCH(st, hipLaunchKernelGGL((k_init_pops<ST>), dim3((unsigned)blocks), dim3(256), 0,
                                      stream, s, plate, e0, w0));
  return hipGetLastError();
}

hipError_t launch_fields(int st, const DevState &s, int plate, int64_t nodes, int b, double *e,
                         double *w, double *u, double *v, hipStream_t stream) {
  int64_t blocks = (nodes + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  LBM_DISPATCH(st, hipLaunchKernelGGL((k_fields<ST>), dim3((unsigned)blocks), dim3(256), 0,
                                      stream, s, plate, b, e, w, u, v));
  return hipGetLastError();
}

hipError_t launch_cons_err(int st, const DevState &s, int plate, int64_t nodes, int b, double *err,
                           hipStream_t stream) {
  int64_t blocks = (nodes + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  LBM_DISPATCH(st, hipLaunchKernelGGL((k_cons_err<ST>), dim3((unsigned)blocks), dim3(256), 0,
                                      stream, s, plate, b, err));
  return hipGetLastError();
}

// ------------------------------------------- fixed staging of lbm_fields_noalloc
//
// Device memory of the library's own, for callers that cannot allocate: a
// file-scope array that every context on a GPU shares (each GPU holds its
// own copy, at its own address, until the process ends).  Host code never
// passes the array's name to a kernel or a copy (on the host it only stands
// for the symbol); it uses the device address hipGetSymbolAddress returns,
// looked up once per device with that device current.
static __device__ __align__(256) double scratch[kNoAllocBytes / sizeof(double)];

namespace {
std::mutex g_scratch_mu;
constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices] = {};
hipError_t g_scratch_err[kMaxDevices] = {};
bool g_scratch_done[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_staging(int device, void **ptr) {
  *ptr = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_done[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch_err[device] = e;
    g_scratch_ptr[device] = e == hipSuccess ? p : nullptr;
    g_scratch_done[device] = true;
  }
  *ptr = g_scratch_ptr[device];
  return g_scratch_err[device];
}

}  // namespace lbm
