// Host-only check of the block pass's patches (no GPU): cuts plates read from
// stdin with the library's host code and checks what the kernel relies on.
// Built by tests/test_patches_cpu.py; the class bytes and boundary records
// come from the library's host source, whose kernel launchers are stubs.
//
// stdin: n_plates, then per plate: nx ny periodic_x periodic_y, ny rows of
//        nx 0/1; n_plans, then per plan: steps, rows per wave, rows
//        of a patch without boundary nodes, 1 for reading R2
// stdout: per plan "patches P bounded B tasks T violations V"
#include <cstdio>
#include <iostream>
#include <string>
#include <vector>

#define main tiles_main
#include "tiles_harness.cpp"
#undef main

int main() {
  int np;
  if (!(std::cin >> np)) return 2;
  std::vector<PlateHost> ph(np);
  std::vector<std::vector<BndNode>> bnd(np);
  std::vector<std::vector<uint8_t>> masks(np);
  for (int p = 0; p < np; p++) {
    lbm_plate pl{};
    int px, py;
    std::cin >> pl.nx >> pl.ny >> px >> py;
    masks[p].resize((size_t)pl.nx * pl.ny);
    for (auto &m : masks[p]) {
      int v;
      std::cin >> v;
      m = (uint8_t)v;
    }
    pl.mask = masks[p].data();
    pl.periodic_x = (uint8_t)px;
    pl.periodic_y = (uint8_t)py;
    ph[p].nx = pl.nx;
    ph[p].ny = pl.ny;
    ph[p].px = px != 0;
    ph[p].py = py != 0;
    std::string why;
    if (!classify(pl, ph[p], why)) {
      printf("classify: %s\n", why.c_str());
      return 3;
    }
    for (int j = 0; j < pl.ny; j++)
      for (int i = 0; i < pl.nx; i++)
        if (ph[p].cls[(size_t)j * pl.nx + i] & CL_B) {
          BndNode b{};
          b.i = i;
          b.j = j;
          bnd[p].push_back(b);
        }
  }
  std::vector<PatchPlate> pp(np);
  int64_t b0 = 0;
  for (int p = 0; p < np; p++) {
    pp[p].index = p;
    pp[p].nx = ph[p].nx;
    pp[p].ny = ph[p].ny;
    pp[p].px = ph[p].px;
    pp[p].py = ph[p].py;
    pp[p].cls = ph[p].cls.data();
    pp[p].bnd = bnd[p].data();
    pp[p].nb = (int64_t)bnd[p].size();
    pp[p].b0 = b0;
    b0 += pp[p].nb;
  }
  int nplans, total = 0;
  std::cin >> nplans;
  for (int q = 0; q < nplans; q++) {
    int K, rows, inner, streamed, bad = 0, bounded = 0;
    std::cin >> K >> rows >> inner >> streamed;
    for (auto &p : pp) p.streamed = streamed != 0;
    PatchPlan plan;
    if (!make_patch_plan(pp, K, rows, inner, plan)) {
      printf("plan %d %d %d: not cut\n", K, rows, inner);
      total++;
      continue;
    }
    const size_t nb = plan.patches.size();  // (then the patches without boundary nodes)
    plan.patches.insert(plan.patches.end(), plan.inner.begin(), plan.inner.end());
    auto report = [&](const char *what, size_t i) {
      if (bad++ < 10) {
        const Patch &t = plan.patches[i];
        printf("violation: %s: patch %zu of plate %d at (%d, %d) %d x %d\n", what, i, t.plate, t.ex, t.ey,
               t.ew, t.eh);
      }
    };
    std::vector<std::vector<uint8_t>> owner(np);
    for (int p = 0; p < np; p++) owner[p].assign(ph[p].cls.size(), 0);
    for (size_t i = 0; i < plan.patches.size(); i++) {
      const Patch &t = plan.patches[i];
      const PlateHost &h = ph[t.plate];
      const bool has = t.b1 > t.b0;
      bounded += has;
      if (has != (i < nb)) report("list", i);
      const int hmax = has ? rows * (kBlockThreads / 64 - 1) * (kBlockCols / t.w) : inner;
      if (t.w != kBlockCols && (t.w != kBlockCols / 2 || !has)) report("shape", i);
      if (t.ew < 1 || t.ew > t.w || t.eh < 1 || t.eh > hmax) report("size", i);
      if (t.ox0 < 0 || t.ox1 > t.ew || t.ox0 >= t.ox1 || t.oy0 < 0 || t.oy1 > t.eh || t.oy0 >= t.oy1)
        report("owned rectangle", i);
      if (t.b1 - t.b0 > kBlockTasks) report("tasks", i);
      if (!h.px && (t.ex < 0 || t.ex + t.ew > h.nx)) report("past a bounded x edge", i);
      if (!h.py && (t.ey < 0 || t.ey + t.eh > h.ny)) report("past a bounded y edge", i);
      auto cls = [&](int a, int b) -> uint8_t {  // patch coordinates; 0 outside the patch
        if (a < 0 || a >= t.ew || b < 0 || b >= t.eh) return 0;
        const int x = ((t.ex + a) % h.nx + h.nx) % h.nx, y = ((t.ey + b) % h.ny + h.ny) % h.ny;
        return h.cls[(size_t)y * h.nx + x];
      };
      for (int b = t.oy0; b < t.oy1; b++)
        for (int a = t.ox0; a < t.ox1; a++) {
          const int x = ((t.ex + a) % h.nx + h.nx) % h.nx, y = ((t.ey + b) % h.ny + h.ny) % h.ny;
          owner[t.plate][(size_t)y * h.nx + x]++;
        }
      if (t.g1 - t.g0 > kBlockGrads) report("gradient nodes", i);
      // the tasks: every boundary node of the patch, with its record and
      // place, and the gradient nodes of itself and its body neighbours
      int at = t.b0;
      for (int b = 0; b < t.eh; b++)
        for (int a = 0; a < t.ew; a++) {
          const uint8_t c = cls(a, b);
          if (!(c & CL_B)) continue;
          if (!has) {
            report("boundary node in a patch without tasks", i);
            continue;
          }
          const PTask &T = plan.tasks[(size_t)at];
          const BndNode &B = bnd[t.plate][(size_t)(T.bnd - pp[t.plate].b0)];
          const int x = ((t.ex + a) % h.nx + h.nx) % h.nx, y = ((t.ey + b) % h.ny + h.ny) % h.ny;
          const bool own = a >= t.ox0 && a < t.ox1 && b >= t.oy0 && b < t.oy1;
          if (T.l != b * t.w + a || B.i != x || B.j != y || (T.own != 0) != own) report("task", i);
          const int di[5] = {0, 1, 0, -1, 0}, dj[5] = {0, 0, 1, 0, -1};
          for (int d = 0; d < 5; d++) {
            const bool in = (cls(a + di[d], b + dj[d]) & CL_IN) != 0;
            if (in != (T.g[d] >= 0)) report("gradient of a neighbour", i);
            if (!in || T.g[d] < 0) continue;
            if (T.g[d] >= t.g1 - t.g0) {
              report("gradient index", i);
              continue;
            }
            const PGrad &G = plan.grads[(size_t)(t.g0 + T.g[d])];
            const int xx = ((x + di[d]) % h.nx + h.nx) % h.nx, yy = ((y + dj[d]) % h.ny + h.ny) % h.ny;
            if (G.l != (b + dj[d]) * t.w + a + di[d]) report("gradient place", i);
            if (G.code != (fd_code_host(h, xx, yy, 0) | (fd_code_host(h, xx, yy, 1) << 3)))
              report("stencil code", i);
            if (d == 0 && G.task != at - t.b0) report("gradient's task", i);
          }
          at++;
        }
      if (at != t.b1) report("task count", i);
      for (int g = t.g0; g < t.g1; g++) {
        const PGrad &G = plan.grads[(size_t)g];
        const uint8_t c = cls(G.l % t.w, G.l / t.w);
        if (!(c & CL_IN) || (G.task >= 0) != ((c & CL_B) != 0)) report("gradient node", i);
      }
      // K steps of validity: a value is valid if everything it is computed
      // from is (nothing is known outside the patch); the owned nodes must be
      const int n = t.ew * t.eh;
      std::vector<uint8_t> F(n), U(n), F1(n), U1(n);
      for (int b = 0; b < t.eh; b++)
        for (int a = 0; a < t.ew; a++) F[b * t.ew + a] = U[b * t.ew + a] = (cls(a, b) & CL_IN) != 0;
      auto get = [&](const std::vector<uint8_t> &v, int a, int b) {
        return a >= 0 && a < t.ew && b >= 0 && b < t.eh && v[(size_t)(b * t.ew + a)];
      };
      const int di[4] = {1, 0, -1, 0}, dj[4] = {0, 1, 0, -1};
      const uint8_t nbit[4] = {NB_E, NB_N, NB_W, NB_S};
      auto stencil = [&](const std::vector<uint8_t> &v, int a, int b) {
        if (!get(v, a, b)) return false;
        const int x = ((t.ex + a) % h.nx + h.nx) % h.nx, y = ((t.ey + b) % h.ny + h.ny) % h.ny;
        for (int ax = 0; ax < 2; ax++) {
          const int dx = ax == 0, dy = ax != 0;
          const int c = fd_code_host(h, x, y, ax);
          if (c == FD_CENTRAL && !(get(v, a + dx, b + dy) && get(v, a - dx, b - dy))) return false;
          if ((c == FD_FWD3 || c == FD_FWD2) && !get(v, a + dx, b + dy)) return false;
          if ((c == FD_BWD3 || c == FD_BWD2) && !get(v, a - dx, b - dy)) return false;
          if (c == FD_FWD3 && !get(v, a + 2 * dx, b + 2 * dy)) return false;
          if (c == FD_BWD3 && !get(v, a - 2 * dx, b - 2 * dy)) return false;
        }
        return true;
      };
      for (int s = 0; s < K; s++) {
        for (int b = 0; b < t.eh; b++)
          for (int a = 0; a < t.ew; a++) {
            const uint8_t c = cls(a, b);
            bool ok = (c & CL_IN) && get(U, a, b);
            if (ok && (c & CL_B)) {
              ok = stencil(U, a, b);
              for (int d = 0; d < 4; d++)
                if (c & nbit[d]) ok = ok && stencil(U, a + di[d], b + dj[d]);
            } else if (ok) {
              for (int d = 0; d < 4; d++) ok = ok && get(F, a + di[d], b + dj[d]);
            }
            U1[(size_t)(b * t.ew + a)] = ok;
          }
        for (int pass = 0; pass < 2; pass++)  // boundary nodes first
          for (int b = 0; b < t.eh; b++)
            for (int a = 0; a < t.ew; a++) {
              const uint8_t c = cls(a, b);
              if (((c & CL_B) != 0) != (pass == 0)) continue;
              bool ok = (c & CL_IN) != 0;
              if (ok && (c & CL_B)) {
                ok = stencil(U1, a, b);
                for (int d = 0; d < 4; d++)
                  if (streamed && (c & nbit[d])) ok = ok && get(F, a + di[d], b + dj[d]);
              } else if (ok) {
                ok = get(F, a, b);
                for (int d = 0; d < 4; d++) {
                  ok = ok && get(F, a + di[d], b + dj[d]);
                  if (cls(a + di[d], b + dj[d]) & CL_B) ok = ok && get(F1, a + di[d], b + dj[d]);
                }
              }
              F1[(size_t)(b * t.ew + a)] = ok;
            }
        F.swap(F1);
        U.swap(U1);
      }
      for (int b = t.oy0; b < t.oy1; b++)
        for (int a = t.ox0; a < t.ox1; a++)
          if ((cls(a, b) & CL_IN) && !(get(F, a, b) && get(U, a, b))) report("owned node lacks a dependence", i);
    }
    for (int p = 0; p < np; p++)
      for (size_t k = 0; k < owner[p].size(); k++)
        if (owner[p][k] > 1 || ((ph[p].cls[k] & CL_IN) && owner[p][k] != 1)) {
          if (bad++ < 10)
            printf("violation: node %zu of plate %d owned %d times\n", k, p, (int)owner[p][k]);
        }
    printf("patches %zu bounded %d tasks %zu violations %d\n", plan.patches.size(), bounded,
           plan.tasks.size(), bad);
    total += bad;
  }
  return total ? 1 : 0;
}
