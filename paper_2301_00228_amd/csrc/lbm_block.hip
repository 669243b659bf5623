// lbm_block.hip -- several time steps of a patch per pass (gfx950).
//
// A block pass advances every plate by up to K steps.  A workgroup owns a
// rectangle of nodes and holds it, with the halo its K steps depend on, in
// registers: lane = column (64 of them), each wave M consecutive rows, every
// node's populations and u, du/dt in its lane.  All steps are taken there --
// collide, pull, acceleration, update of u, the boundary reset, the second-row
// rule and the boundary accelerations -- and only the owned nodes of t + K are
// written.  What the halo's outer nodes compute after their neighbourhood is
// missing never reaches an owned node (the host derives the halo from the
// method's dependences).
//
// Neighbours: along x through wave shifts (no LDS), along y in the lane's own
// registers, across row groups through one LDS row per group and side.
//
// k_block takes the patches with boundary nodes, and all patches of small
// plates: eight waves, one workgroup per CU.  In a patch with boundary nodes u
// is kept in LDS; every thread takes at most one node whose gradient the
// boundary needs (a boundary node's thread goes on to its reset field and to the
// population its second-row neighbours pull, eq. LBE_mod; one value per field,
// since J = 0 at boundary nodes under reading R1 and the four moving populations
// are equal), and the eighth wave takes the boundary accelerations from the
// gradient nodes' stresses, one lane per node, beside the seven others' march.
// (With the whole boundary work in that one wave, five gradients per node, a
// step of a patch with boundary nodes took 11 us instead of 2.)  A step depends
// on two nodes along a boundary and one across it, so a patch along an x edge is
// tall: 32 columns, two row groups side by side in each wave, twice the rows (as
// wide ones such patches owned 4 to 11 rows each of 28 to 42; 1024^2 was cut
// into 418 patches with boundary nodes, now 146, 256 plates 3564 per 16, now 1212).
//
// Plates of other readings (VAR) take the same patches: the flux of eq.
// correction-f that streams into a boundary node comes from the march, the node's
// thread keeps its stored populations and leaves one pulled population per
// direction.  (With one interior and one boundary launch per step 257^2 FP64 took
// 30 us per step, now 6.8.)
//
// k_inner takes the other patches of large plates with four waves and up to 256
// registers per lane, so that two workgroups share a CU and one's loads and
// stores run beside the other's steps (one workgroup of eight waves loaded and
// computed in turn).  On small plates without boundary nodes it takes short
// patches (eight waves of two rows): a step there takes as long as the rows of
// a CU, 0.4 us each in FP64.
//
// Why: one launch per step costs 14 us on the smallest plates whatever their
// size (launch gap, then a serial chain of dependent memory reads), and a
// large plate moves its whole state every step; here a step costs one to
// three barriers and no memory traffic.  Measured, us per step, one launch per
// step -> k_block alone with K = 4 -> now: 64^2 periodic FP64 14.1 -> 3.6 -> 1.9,
// 97^2 with loads 14.0 -> 6.1 -> 4.7, 1024^2 clamped 51 -> 20 -> 17, 4096^2 with
// a hole 805 -> 289 -> 205, FP32 450 -> 163 -> 104, F16DEV 474 -> 222 -> 127.
// Small plates are bound by the pass's latency (launch, one load, the steps'
// chains); k_inner by memory in FP64 (8192^2 with a hole, counted: 10.0 GB read,
// 1.40 times the state, and 7.3 written per pass at 4.76 TB/s, 0.92 of a copy of the
// state's arrays) and mostly in F32DEV (5.7 and 4.9 GB, 1.24 times the state, at 4.34
// TB/s, 0.84), in FP32 by both that and the vector units (86 operations per
// node and step, 85 % busy), in the 16-bit storages by their rounding (137).
//
// A step's chain is kept short by what does not change from step to step: a
// gradient node's stencil (its two neighbours and coefficients per axis) and a
// second-row node's upwind boundary nodes are looked up once per pass, and the
// pull asks per row and direction, wave-uniformly, whether any lane has one.
// (Looked up in every step they took 1.5k to 4.3k cycles of about 8k; 97^2
// with loads 6.9 us per step, 1024^2 in F32 16.)
#include <hip/hip_runtime.h>

#include "../../include/lbm.h"
#include "lbm_device.h"
#include "lbm_kernels.h"
#include "lbm_types.h"

namespace lbm {
namespace {

constexpr int kWaves = kBlockThreads / 64;

// The value of lane - 1 (from_west) / lane + 1 (from_east); 0 past the end.
__device__ __forceinline__ int lane_shift_w(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int lane_shift_e(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ float from_west(float v) { return __int_as_float(lane_shift_w(__float_as_int(v))); }
__device__ __forceinline__ float from_east(float v) { return __int_as_float(lane_shift_e(__float_as_int(v))); }
__device__ __forceinline__ double from_west(double v) {
  return __hiloint2double(lane_shift_w(__double2hiint(v)), lane_shift_w(__double2loint(v)));
}
__device__ __forceinline__ double from_east(double v) {
  return __hiloint2double(lane_shift_e(__double2hiint(v)), lane_shift_e(__double2loint(v)));
}

// Per field of a boundary node: the reset field and the population pulled
// from it (VAR: some plate uses readings other than R1 and M1; the flux of eq.
// correction-f is then not 0 and each neighbour pulls another population).
template <class C, bool VAR>
struct BndOut {
  C fld[2], pull[2];
};
template <class C>
struct BndOut<C, true> {
  C fld[2], pull[2][4], j[2][2];
};
// State of a boundary node between steps: u, du/dt, and its boundary data.
template <class U>
struct BndState {
  U u[4];
  double val[2];  // (FP64 whatever U: the amplitude multiplies it in FP64)
  U cell[5];
  int32_t kind, load;
};

template <class U>
struct alignas(2 * sizeof(U)) Vec2 {
  U x, y;
};

// [step parity][0: a row group's first row, 1: its last row][rho phi, rho psi,
// population leaving across that row phi, psi][group * w + column]
template <class CD, int W>
struct EdgeLds {
  typename CD::C edge[2][2][4][64 * W];
};

template <class CD, int M, bool VAR>
struct BlockLds : EdgeLds<CD, kWaves> {
  using C = typename CD::C;
  using U = typename CD::U;
  // patches with boundary nodes (seven interior waves)
  Vec2<U> u[64 * M * (kWaves - 1)];      // displacement of the patch
  uint16_t task[64 * M * (kWaves - 1)];  // boundary task of a node + 1, 0 elsewhere
  PTask rec[kBlockTasks];
  BndState<U> st[kBlockTasks];
  U stress[kBlockGrads][3];
  BndOut<C, VAR> out[kBlockTasks];
};

// One axis of a finite-difference stencil at patch node l, from its code:
// ((c[0] q + c[1] qa) + c[2] qb) times 1/(2 dh) or 1/dh, with q at l, qa, qb at
// a, b (the coefficients of fd_vals; small integers, so kept in FP32).  Nodes
// whose stencil leaves the patch are never needed; their indices are clamped.
struct AxisStencil {
  int a, b;
  float c[3];
  bool half;  // 1/(2 dh)
  __device__ __forceinline__ void set(int code, int l, int d, int last) {
    const bool cen = code == FD_CENTRAL, f3 = code == FD_FWD3, b3 = code == FD_BWD3;
    const bool f2 = code == FD_FWD2, b2 = code == FD_BWD2;
    a = l + ((cen || f3 || f2) ? d : (b3 || b2) ? -d : 0);
    b = l + (cen ? -d : f3 ? 2 * d : b3 ? -2 * d : 0);
    a = a < 0 ? 0 : a > last ? last : a;
    b = b < 0 ? 0 : b > last ? last : b;
    c[0] = f3 ? -3.0f : b3 ? 3.0f : f2 ? -1.0f : b2 ? 1.0f : 0.0f;
    c[1] = (cen || f2) ? 1.0f : f3 ? 4.0f : b3 ? -4.0f : b2 ? -1.0f : 0.0f;
    c[2] = (cen || f3) ? -1.0f : b3 ? 1.0f : 0.0f;
    half = cen || f3 || b3;
  }
  template <class U>
  __device__ __forceinline__ void apply(const Vec2<U> *us, const Vec2<U> &q, const PlateDev &P, U &dx,
                                        U &dy) const {
    const Vec2<U> qa = us[a], qb = us[b];
    const U c0 = (U)c[0], ca = (U)c[1], cb = (U)c[2], sc = half ? (U)P.inv_2h : (U)P.inv_h;
    dx = ((c0 * q.x + ca * qa.x) + cb * qb.x) * sc;
    dy = ((c0 * q.y + ca * qa.y) + cb * qb.y) * sc;
  }
};

// The gradient node of a thread (patches with boundary nodes) and, if that is
// a boundary node, its rest and moving population of the previous step (VAR: its
// stored populations).
template <class CD, bool VAR>
struct GradDuty {
  using C = typename CD::C;
  using U = typename CD::U;
  using Slot = typename CD::Slot;
  int l = -1, task = -1;
  AxisStencil sx, sy;
  C fo[2][2];
  Slot old[2][5];

  __device__ __forceinline__ void load(const DevState &s, const BlockArgs &a, const Patch &t,
                                       const PlateDev &P, int last) {
    if ((int)threadIdx.x >= t.g1 - t.g0) return;
    const PGrad G = a.grads[t.g0 + (int)threadIdx.x];
    l = G.l;
    sx.set(G.code & 7, l, 1, last);
    sy.set((G.code >> 3) & 7, l, t.w, last);
    task = G.task;
    if (task < 0) return;
    const int64_t k = s.bnd[a.tasks[t.b0 + task].bnd].node;
#pragma unroll
    for (int fl = 0; fl < 2; fl++) {
      C f[5];
      CD::load_raw(s, a.in, fl, k, old[fl]);
      CD::raw_to_pops(P, fl, old[fl], f);
      fo[fl][0] = f[0];
      fo[fl][1] = f[1];
    }
  }

  // Stress at the node from u in LDS and, if reset, a boundary node's reset
  // fields and f~ -- the average of its populations of this step and the
  // previous one -- collided towards its own equilibrium (eq. LBE_mod; J = 0).
  template <class L>
  __device__ __forceinline__ void run(const PlateDev &P, L &lds, bool reset) {
    if (l < 0) return;
    U g[4], sg[3];  // d_x u_x, d_y u_x, d_x u_y, d_y u_y
    const Vec2<U> q0 = lds.u[l];
    sx.apply(lds.u, q0, P, g[0], g[2]);
    sy.apply(lds.u, q0, P, g[1], g[3]);
    hooke<U>(P, g, sg[0], sg[1], sg[2]);
#pragma unroll
    for (int q = 0; q < 3; q++) lds.stress[threadIdx.x][q] = sg[q];
    if (!reset || task < 0) return;
    if constexpr (VAR) {
      reset_by_readings(P, lds, g);
      return;
    } else {
    BndOut<C, VAR> o;
#pragma unroll
    for (int fl = 0; fl < 2; fl++) {
      o.fld[fl] = fl == 0 ? (C)(g[0] + g[3]) : (C)(g[2] - g[1]);
      C fn[5], f[5], r, fc[5];
      CD::eq_pops(P, fl, o.fld[fl], C(0), C(0), fn);
      f[0] = C(0.5) * (fn[0] + fo[fl][0]);
#pragma unroll
      for (int q = 1; q < 5; q++) f[q] = C(0.5) * (fn[q] + fo[fl][1]);
      collide_pops<CD>(P, fl, f, r, fc);
      o.pull[fl] = fc[1];
      fo[fl][0] = fn[0];
      fo[fl][1] = fn[1];
    }
    lds.out[task] = o;
    }
  }

  // The same under the plate's readings (see pull_from_boundary in
  // lbm_kernels.hip): R2 takes the flux the march has left in lds.out, R1 that of
  // the previous populations; M2 collides with their equilibrium.
  template <class L>
  __device__ __forceinline__ void reset_by_readings(const PlateDev &P, L &lds, const U g[4]) {
    BndOut<C, true> &o = lds.out[task];
#pragma unroll
    for (int fl = 0; fl < 2; fl++) {
      const C fld = fl == 0 ? (C)(g[0] + g[3]) : (C)(g[2] - g[1]);
      C jox, joy, fn[5], f[5], e[5];
      CD::raw_flux(old[fl], jox, joy);
      const bool streamed = P.readings & RD_FLUX_STREAMED;
      const C jx = streamed ? o.j[fl][0] : jox, jy = streamed ? o.j[fl][1] : joy;
      CD::eq_pops(P, fl, fld, jx, jy, fn);
      CD::raw_to_pops(P, fl, old[fl], f);
#pragma unroll
      for (int q = 0; q < 5; q++) f[q] = C(0.5) * (fn[q] + f[q]);
      if (P.readings & RD_EQ_OLD) {
        CD::eq_pops(P, fl, CD::raw_rho(old[fl]), jox, joy, e);
#pragma unroll
        for (int q = 1; q < 5; q++) o.pull[fl][q - 1] = f[q] - C(2.0) * (f[q] - e[q]);
      } else {
        C r;
        collide_pops<CD>(P, fl, f, r, e);
#pragma unroll
        for (int q = 1; q < 5; q++) o.pull[fl][q - 1] = e[q];
      }
      o.fld[fl] = fld;
      o.j[fl][0] = jx;
      o.j[fl][1] = jy;
      CD::eq_raw(P, fl, fld, jx, jy, old[fl]);
    }
  }
};

// The boundary accelerations of a patch, by its last wave; the barriers are
// those of block_march<BND>.
template <class CD, int M, bool VAR>
__device__ __forceinline__ void block_boundary(const DevState &s, const BlockArgs &a, const Patch &t,
                                               const PlateDev &P, BlockLds<CD, M, VAR> &lds) {
  using U = typename CD::U;
  constexpr int kLast = 64 * M * (kWaves - 1) - 1;
  const int lane = threadIdx.x & 63;
  const int nb = t.b1 - t.b0;
  const unsigned long long n0 = s.counter[a.in];
  GradDuty<CD, VAR> duty;
  duty.load(s, a, t, P, kLast);
  for (int i = lane; i < nb; i += 64) {
    const PTask T = a.tasks[t.b0 + i];
    const BndNode B = s.bnd[T.bnd];
    BndState<U> S;
    S.u[0] = ldg<U>(s.u[a.in][0], B.node);
    S.u[1] = ldg<U>(s.u[a.in][1], B.node);
    S.u[2] = ldg<U>(s.v[a.in][0], B.node);
    S.u[3] = ldg<U>(s.v[a.in][1], B.node);
    S.val[0] = B.val[0];
    S.val[1] = B.val[1];
#pragma unroll
    for (int q = 0; q < 5; q++) S.cell[q] = (U)B.cell[q];
    S.kind = B.kind;
    S.load = B.load;
    lds.rec[i] = T;
    lds.st[i] = S;
  }
  __syncthreads();  // (u in LDS, task map cleared)
  for (int i = lane; i < nb; i += 64) lds.task[lds.rec[i].l] = (uint16_t)(i + 1);
  duty.run(P, lds, false);
  __syncthreads();
  for (int j = 0; j < a.steps; j++) {
    const unsigned long long n = n0 + (unsigned long long)j;
    const Kick<U> kick = kick_of<U>(P, n == 0);
    // accelerations at t_n; u, du/dt of t_{n+1} (nothing reads u in LDS here)
    for (int i = lane; i < nb; i += 64) {
      const PTask T = lds.rec[i];
      BndState<U> &S = lds.st[i];
      const U ux = S.u[0], uy = S.u[1], vx = S.u[2], vy = S.u[3];
      U ax, ay;
      if (S.kind == LBM_BC_DIRICHLET) {
        const double g = load_amp(s, S.load, (double)(n + 1) * P.dt);
        dirichlet_accel<U>(P, n, (U)(g * S.val[0]), (U)(g * S.val[1]), ux, uy, vx, vy, ax, ay);
      } else {
        const double g = load_amp(s, S.load, (double)n * P.dt);
        U sk[3], sr[4][3];
        bool has[4];
#pragma unroll
        for (int q = 0; q < 3; q++) sk[q] = lds.stress[T.g[0]][q];
#pragma unroll
        for (int d = 0; d < 4; d++) {
          has[d] = T.g[1 + d] >= 0;
          const int gi = has[d] ? T.g[1 + d] : T.g[0];
#pragma unroll
          for (int q = 0; q < 3; q++) sr[d][q] = lds.stress[gi][q];
        }
        const U l4[4] = {S.cell[1], S.cell[2], S.cell[3], S.cell[4]};
        neumann_accel<U>(P, sk, has, sr, S.cell[0], l4, (U)(g * S.val[0]), (U)(g * S.val[1]), ax,
                         ay);
      }
      U q[4];
      newmark<U>(P, kick, ax, ay, ux, uy, vx, vy, q[0], q[1], q[2], q[3]);
#pragma unroll
      for (int c = 0; c < 4; c++) S.u[c] = q[c];
      lds.u[T.l] = Vec2<U>{q[0], q[1]};
      if (T.own && (!(fabs((double)q[0]) < 1e30) || !(fabs((double)q[1]) < 1e30))) s.flag[0] = 1;
    }
    __syncthreads();
    __syncthreads();
    duty.run(P, lds, true);
    __syncthreads();
  }
  for (int i = lane; i < nb; i += 64)
    if (lds.rec[i].own) {
      const int64_t k = s.bnd[lds.rec[i].bnd].node;
      stg<U>(s.u[a.out][0], k, lds.st[i].u[0]);
      stg<U>(s.u[a.out][1], k, lds.st[i].u[1]);
      stg<U>(s.v[a.out][0], k, lds.st[i].u[2]);
      stg<U>(s.v[a.out][1], k, lds.st[i].u[3]);
    }
}

// The interior waves of a patch; BND: it holds boundary nodes (the last wave
// is block_boundary's).
template <class CD, int M, int kW, bool BND, bool VAR, class Lds>
__device__ __forceinline__ void block_march(const DevState &s, const BlockArgs &a, const Patch &t,
                                            const PlateDev &P, Lds &lds) {
  using C = typename CD::C;
  using U = typename CD::U;
  using Slot = typename CD::Slot;
  constexpr int kLast = 64 * M * kW - 1;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const unsigned long long n0 = s.counter[a.in];

  // ---- the state of t: row r = wv M + m of the patch, column lane (lanes and
  // rows past the patch repeat its last one)
  auto wrap = [](int i, int n) { return i < 0 || i >= n ? ((i % n) + n) % n : i; };
  // (the row groups of M rows: one per wave, two in a patch of w = 32 columns)
  const int w = BND ? t.w : 64;
  const int col = lane & (w - 1), grp = BND ? (int)(threadIdx.x / (unsigned)w) : wv;
  const int at0 = grp * M * w + col;  // place of the lane's first node in the patch
  // (what a pass of fewer steps does not depend on repeats nodes that it does)
  const int h = BND ? kBlockCols : a.steps;
  const int x0 = t.ox0 > h ? t.ox0 - h : 0, x1 = t.ox1 + h < t.ew ? t.ox1 + h : t.ew;
  const int y0 = t.oy0 > h ? t.oy0 - h : 0, y1 = t.oy1 + h < t.eh ? t.oy1 + h : t.eh;
  auto within = [](int i, int lo, int hi) { return i < lo ? lo : i < hi ? i : hi - 1; };
  const int x = wrap(t.ex + within(col, x0, x1), P.nx);
  auto node = [&](int m) { return node_of(P, x, wrap(t.ey + within(grp * M + m, y0, y1), P.ny)); };
  // (away from boundary nodes only a node's own update reads its u and du/dt:
  // the halo's lanes repeat an owned node's)
  const int xo = wrap(t.ex + within(col, t.ox0, t.ox1), P.nx);
  auto own_node = [&](int m) {
    return node_of(P, xo, wrap(t.ey + within(grp * M + m, t.oy0, t.oy1), P.ny));
  };
  auto mine = [&](int m) {
    const int r = grp * M + m;
    return col >= t.ox0 && col < t.ox1 && r >= t.oy0 && r < t.oy1;
  };
  GradDuty<CD, VAR> duty;
  if constexpr (BND) duty.load(s, a, t, P, kLast);
  // task + 1 (0: none) of a boundary node (low half of up[0]) or of a second-row
  // node's upwind boundary nodes W, S, E, N; which (row, direction) any lane of
  // the wave has, and which rows hold boundary nodes
  uint32_t up[M][2], some = 0, some_b = 0;
#pragma unroll
  for (int m = 0; m < M; m++) up[m][0] = up[m][1] = 0;
  uint8_t cl[M];
  Slot raw[M][2][5];
  U uv[M][4];
#pragma unroll
  for (int m = 0; m < M; m++) {
    const int64_t k = node(m);
    cl[m] = BND ? s.cls[k] : (uint8_t)CL_IN;
    CD::load_raw(s, a.in, 0, k, raw[m][0]);
    CD::load_raw(s, a.in, 1, k, raw[m][1]);
    const int64_t ku = BND ? k : own_node(m);
    uv[m][0] = ldg<U>(s.u[a.in][0], ku);
    uv[m][1] = ldg<U>(s.u[a.in][1], ku);
    uv[m][2] = ldg<U>(s.v[a.in][0], ku);
    uv[m][3] = ldg<U>(s.v[a.in][1], ku);
  }
  if constexpr (BND) {
#pragma unroll
    for (int m = 0; m < M; m++) {
      const int l = at0 + m * w;
      if (col >= t.ew || grp * M + m >= t.eh) cl[m] = 0;
      lds.u[l] = Vec2<U>{uv[m][0], uv[m][1]};
      lds.task[l] = 0;
      if (!(cl[m] & CL_IN)) {
#pragma unroll
        for (int fl = 0; fl < 2; fl++)
#pragma unroll
          for (int q = 0; q < 5; q++) raw[m][fl][q] = Slot(0);
      }
    }
    __syncthreads();
    duty.run(P, lds, false);
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; m++) {
      const int l = at0 + m * w;
      // (a node past the patch has no task, and no needed node has one there)
      auto task_at = [&](int k) { return k < 0 || k > kLast ? 0u : (uint32_t)lds.task[k]; };
      if (cl[m] & CL_B) up[m][0] = task_at(l);
      if (cl[m] & CL_S) {
        up[m][0] = task_at(l - 1) | task_at(l - w) << 16;
        up[m][1] = task_at(l + 1) | task_at(l + w) << 16;
      }
      some |= (uint32_t)(__any((cl[m] & CL_S) && (up[m][0] & 0xffffu)) ? 1 : 0) << (4 * m);
      some |= (uint32_t)(__any((cl[m] & CL_S) && (up[m][0] >> 16)) ? 2 : 0) << (4 * m);
      some |= (uint32_t)(__any((cl[m] & CL_S) && (up[m][1] & 0xffffu)) ? 4 : 0) << (4 * m);
      some |= (uint32_t)(__any((cl[m] & CL_S) && (up[m][1] >> 16)) ? 8 : 0) << (4 * m);
      some_b |= (uint32_t)(__any((cl[m] & CL_B) != 0) ? 1 : 0) << m;
    }
  }

  for (int j = 0; j < a.steps; j++) {
    const Kick<U> kick = kick_of<U>(P, n0 + (unsigned long long)j == 0);
    const int par = j & 1;
    // ---- collide; interior acceleration, u and du/dt of t_{n+1} of the rows
    // between two of the lane's own (before the exchange: their neighbours' moments
    // then need no registers after it); the first and last row go to the
    // neighbouring groups
    C rho[M][2], fs[M][2][5];
    auto update = [&](int m, const C *ss, const C *nn) {
      const C e0 = from_east(rho[m][0]), w0 = from_west(rho[m][0]);
      const C e1 = from_east(rho[m][1]), w1 = from_west(rho[m][1]);
      U q[4];
      interior_update<U>(P, kick, (U)e0, (U)w0, (U)nn[0], (U)ss[0], (U)e1, (U)w1, (U)nn[1], (U)ss[1],
                         uv[m][0], uv[m][1], uv[m][2], uv[m][3], q[0], q[1], q[2], q[3]);
#pragma unroll
      for (int c = 0; c < 4; c++) uv[m][c] = q[c];
      if constexpr (BND) {
        if ((cl[m] & (CL_IN | CL_B)) == CL_IN) lds.u[at0 + m * w] = Vec2<U>{q[0], q[1]};
      }
    };
#pragma unroll
    for (int m = 0; m < M; m++) {
#pragma unroll
      for (int fl = 0; fl < 2; fl++) CD::collide_raw(P, fl, raw[m][fl], rho[m][fl], fs[m][fl]);
      if (m >= 2) update(m > 0 ? m - 1 : 0, rho[m > 1 ? m - 2 : 0], rho[m]);
    }
#pragma unroll
    for (int fl = 0; fl < 2; fl++) {
      lds.edge[par][0][fl][threadIdx.x] = rho[0][fl];
      lds.edge[par][0][2 + fl][threadIdx.x] = fs[0][fl][4];
      lds.edge[par][1][fl][threadIdx.x] = rho[M - 1][fl];
      lds.edge[par][1][2 + fl][threadIdx.x] = fs[M - 1][fl][2];
    }
    __syncthreads();
    // the rows below and above the group's: their moments, then the populations
    // that come from there
    // (a patch's outermost rows read some finite value: nothing needed depends on it)
    const int ti = (int)threadIdx.x, below = ti >= w ? ti - w : ti, above = ti + w < 64 * kW ? ti + w : ti;
    auto from_below = [&](int q) { return lds.edge[par][1][q][below]; };
    auto from_above = [&](int q) { return lds.edge[par][0][q][above]; };
    {
      const C lo[2] = {from_below(0), from_below(1)}, hi[2] = {from_above(0), from_above(1)};
      update(0, lo, rho[1]);
      update(M - 1, rho[M - 2], hi);
    }
    if constexpr (BND && VAR) {
      // flux of eq. correction-f under reading R2: what streams into a boundary
      // node from its body neighbours
      if (P.readings & RD_FLUX_STREAMED) {
#pragma unroll
        for (int m = 0; m < M; m++) {
          if (!(some_b >> m & 1u)) continue;
#pragma unroll
          for (int fl = 0; fl < 2; fl++) {
            const C fw = from_west(fs[m][fl][1]), fe = from_east(fs[m][fl][3]);
            const C fb = m > 0 ? fs[m > 0 ? m - 1 : 0][fl][2] : from_below(2 + fl);
            const C fa = m + 1 < M ? fs[m + 1 < M ? m + 1 : m][fl][4] : from_above(2 + fl);
            if (!(cl[m] & CL_B) || !up[m][0]) continue;
            C *j2 = lds.out[up[m][0] - 1].j[fl];
            j2[0] = (C(0) + (cl[m] & NB_W ? fw : C(0))) + (cl[m] & NB_E ? -fe : C(0));
            j2[1] = (C(0) + (cl[m] & NB_S ? fb : C(0))) + (cl[m] & NB_N ? -fa : C(0));
          }
        }
      }
    }
    if constexpr (BND) {
      __syncthreads();
      duty.run(P, lds, true);
      __syncthreads();
    }
    // ---- pull: f_alpha(x, t + dt) = f*_alpha(x - c^alpha dt)
    const C lo[2] = {from_below(2), from_below(3)}, hi[2] = {from_above(2), from_above(3)};
#pragma unroll
    for (int m = 0; m < M; m++) {
      C f[2][5];
#pragma unroll
      for (int fl = 0; fl < 2; fl++) {
        f[fl][0] = fs[m][fl][0];
        f[fl][1] = from_west(fs[m][fl][1]);
        f[fl][3] = from_east(fs[m][fl][3]);
        f[fl][2] = m > 0 ? fs[m > 0 ? m - 1 : 0][fl][2] : lo[fl];
        f[fl][4] = m + 1 < M ? fs[m + 1 < M ? m + 1 : m][fl][4] : hi[fl];
      }
      if constexpr (BND) {
        // populations pulled from boundary nodes (eq. LBE_mod)
#pragma unroll
        for (int al = 1; al < 5; al++)
          if (some >> (4 * m + al - 1) & 1u) {
            const uint32_t w2 = up[m][(al - 1) >> 1];
            const uint32_t ti = cl[m] & CL_S ? ((al - 1) & 1 ? w2 >> 16 : w2 & 0xffffu) : 0u;
            const auto &o = lds.out[ti ? ti - 1 : 0];
            C p0, p1;
            if constexpr (VAR) {
              p0 = o.pull[0][al - 1];
              p1 = o.pull[1][al - 1];
            } else {
              p0 = o.pull[0];
              p1 = o.pull[1];
            }
            f[0][al] = ti ? p0 : f[0][al];
            f[1][al] = ti ? p1 : f[1][al];
          }
      }
#pragma unroll
      for (int fl = 0; fl < 2; fl++) CD::encode(P, fl, f[fl], raw[m][fl]);
      if constexpr (BND) {
        if (some_b >> m & 1u) {
          const bool isb = (cl[m] & CL_B) && up[m][0];
          const auto &o = lds.out[isb ? up[m][0] - 1 : 0];
#pragma unroll
          for (int fl = 0; fl < 2; fl++) {
            Slot q5[5];
            if constexpr (VAR)
              CD::eq_raw(P, fl, o.fld[fl], o.j[fl][0], o.j[fl][1], q5);
            else
              CD::eq_raw(P, fl, o.fld[fl], q5);
#pragma unroll
            for (int q = 0; q < 5; q++) raw[m][fl][q] = isb ? q5[q] : raw[m][fl][q];
          }
        }
      }
    }
  }

  // ---- the owned nodes of t + K (u, du/dt of boundary nodes: block_boundary)
#pragma unroll
  for (int m = 0; m < M; m++) {
    if (mine(m) && (cl[m] & CL_IN)) {
      const int64_t k = node(m);
      CD::store_raw(s, a.out, 0, k, raw[m][0]);
      CD::store_raw(s, a.out, 1, k, raw[m][1]);
      if (!BND || !(cl[m] & CL_B)) {
        stg<U>(s.u[a.out][0], k, uv[m][0]);
        stg<U>(s.u[a.out][1], k, uv[m][1]);
        stg<U>(s.v[a.out][0], k, uv[m][2]);
        stg<U>(s.v[a.out][1], k, uv[m][3]);
      }
    }
  }
}

template <int ST, int M, bool VAR = false>
__global__ void __launch_bounds__(kBlockThreads, 2) k_block(DevState s, BlockArgs a) {
  using CD = typename CodecOf<ST>::type;
  __shared__ BlockLds<CD, M, VAR> lds;
  if (a.count && blockIdx.x == 0 && threadIdx.x == 0)
    s.counter[a.out] = s.counter[a.in] + (unsigned long long)a.steps;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);  // (scalar branches)
  const int ix = tile_index(blockIdx.x, a.q);
  if (ix >= a.n) return;
  const Patch t = a.patches[ix];
  const PlateDev P = s.plates[t.plate];
  if (t.b1 <= t.b0)
    block_march<CD, M, kWaves, false, VAR>(s, a, t, P, lds);
  else if (wv < kWaves - 1)
    block_march<CD, M, kWaves - 1, true, VAR>(s, a, t, P, lds);
  else
    block_boundary<CD, M, VAR>(s, a, t, P, lds);
}

// (two waves per SIMD: two workgroups of four waves, or one of eight, per CU)
template <int ST, int M, int W>
__global__ void __launch_bounds__(64 * W, 2) k_inner(DevState s, BlockArgs a) {
  using CD = typename CodecOf<ST>::type;
  __shared__ EdgeLds<CD, W> lds;
  if (a.count && blockIdx.x == 0 && threadIdx.x == 0)
    s.counter[a.out] = s.counter[a.in] + (unsigned long long)a.steps;
  const int ix = tile_index(blockIdx.x, a.q);
  if (ix >= a.n) return;
  const Patch t = a.patches[ix];
  const PlateDev P = s.plates[t.plate];
  block_march<CD, M, W, false, false>(s, a, t, P, lds);
}

template <int ST>
hipError_t launch_block_t(const DevState &s, const BlockArgs &a, int rows, bool var, hipStream_t st) {
  const dim3 grid(8 * a.q), th(kBlockThreads);
  if (var) {
    if (rows != 3) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_block<ST, 3, true>), grid, th, 0, st, s, a);
    return hipGetLastError();
  }
  if (rows == 3) {
    hipLaunchKernelGGL((k_block<ST, 3>), grid, th, 0, st, s, a);
    return hipGetLastError();
  }
  if (rows == 4) {
    hipLaunchKernelGGL((k_block<ST, 4>), grid, th, 0, st, s, a);
    return hipGetLastError();
  }
  if constexpr (ST != LBM_STORE_F64) {  // (FP64: past the registers)
    if (rows == 5) {
      hipLaunchKernelGGL((k_block<ST, 5>), grid, th, 0, st, s, a);
      return hipGetLastError();
    }
    if (rows == 6) {
      hipLaunchKernelGGL((k_block<ST, 6>), grid, th, 0, st, s, a);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}

template <int ST>
hipError_t launch_inner_t(const DevState &s, const BlockArgs &a, int rows, hipStream_t st) {
  constexpr int R = block_inner_rows(ST);
  static_assert(R % 4 == 0 && kInnerSmall % kWaves == 0, "whole rows per wave");
  if (rows == R)
    hipLaunchKernelGGL((k_inner<ST, R / 4, 4>), dim3(8 * a.q), dim3(256), 0, st, s, a);
  else if (rows == kInnerSmall)
    hipLaunchKernelGGL((k_inner<ST, kInnerSmall / kWaves, kWaves>), dim3(8 * a.q), dim3(kBlockThreads), 0,
                       st, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_block(int storage, const DevState &s, const BlockWork &w, int in, int out, int steps,
                        hipStream_t st) {
  if (w.n_patches < 1 || steps < 1) return hipErrorInvalidValue;
  const BlockArgs a{w.patches, w.tasks, w.grads, w.n_patches, (w.n_patches + 7) / 8, in, out, steps, 1};
  switch (storage) {
    case LBM_STORE_F64: return launch_block_t<LBM_STORE_F64>(s, a, w.rows, w.var, st);
    case LBM_STORE_F32: return launch_block_t<LBM_STORE_F32>(s, a, w.rows, w.var, st);
    case LBM_STORE_F32DEV: return launch_block_t<LBM_STORE_F32DEV>(s, a, w.rows, w.var, st);
    case LBM_STORE_F16DEV: return launch_block_t<LBM_STORE_F16DEV>(s, a, w.rows, w.var, st);
    case LBM_STORE_BF16DEV: return launch_block_t<LBM_STORE_BF16DEV>(s, a, w.rows, w.var, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_inner(int storage, const DevState &s, const BlockWork &w, int in, int out, int steps,
                        hipStream_t st) {
  if (w.n_inner < 1 || steps < 1) return hipErrorInvalidValue;
  // (beside a launch_block, that one counts the steps)
  const BlockArgs a{w.inner, nullptr, nullptr, w.n_inner, (w.n_inner + 7) / 8, in, out, steps,
                    w.n_patches < 1};
  switch (storage) {
    case LBM_STORE_F64: return launch_inner_t<LBM_STORE_F64>(s, a, w.inner_rows, st);
    case LBM_STORE_F32: return launch_inner_t<LBM_STORE_F32>(s, a, w.inner_rows, st);
    case LBM_STORE_F32DEV: return launch_inner_t<LBM_STORE_F32DEV>(s, a, w.inner_rows, st);
    case LBM_STORE_F16DEV: return launch_inner_t<LBM_STORE_F16DEV>(s, a, w.inner_rows, st);
    case LBM_STORE_BF16DEV: return launch_inner_t<LBM_STORE_BF16DEV>(s, a, w.inner_rows, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm
