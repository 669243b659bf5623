// Host-only check of the choice of a block pass plan (no GPU): plans plates read
// from stdin with the library's host code.  Built by tests/test_plan_cpu.py; the
// kernel launchers are stubs.
//
// stdin: n_bodies, then per body: storage, readings, nx ny periodic_x periodic_y, ny
//        rows of nx characters 0/1
// stdout: per body "plan use K rows inner patches inner_patches us tiles_us",
//         then per K from 6 to 2 with that plan's rows "K us" (us 0: not cut)
#include <cstdio>
#include <iostream>
#include <string>

#define main tiles_main
#include "tiles_harness.cpp"
#undef main

int main() {
  int nb;
  if (!(std::cin >> nb)) return 2;
  for (int q = 0; q < nb; q++) {
    lbm_ctx c;
    lbm_plate pl{};
    int px, py, readings;
    std::cin >> c.storage >> readings >> pl.nx >> pl.ny >> px >> py;
    std::vector<uint8_t> mask;
    for (int j = 0; j < pl.ny; j++) {
      std::string row;
      std::cin >> row;
      for (char ch : row) mask.push_back(ch == '1');
    }
    if (mask.size() != (size_t)pl.nx * pl.ny) return 2;
    pl.mask = mask.data();
    pl.periodic_x = (uint8_t)px;
    pl.periodic_y = (uint8_t)py;
    c.ph.resize(1);
    c.pd.resize(1);
    PlateHost &h = c.ph[0];
    h.nx = pl.nx;
    h.ny = pl.ny;
    h.px = px != 0;
    h.py = py != 0;
    std::string why;
    if (!classify(pl, h, why)) {
      printf("classify: %s\n", why.c_str());
      return 3;
    }
    c.n_body = h.body;
    c.variant_readings = readings != 0;
    for (int j = 0; j < pl.ny; j++)
      for (int i = 0; i < pl.nx; i++)
        if (h.cls[(size_t)j * pl.nx + i] & CL_B) {
          BndNode b{};
          b.i = i;
          b.j = j;
          c.bnd.push_back(b);
        }
    std::vector<PatchPlate> v(1);
    v[0].nx = h.nx;
    v[0].ny = h.ny;
    v[0].px = h.px;
    v[0].py = h.py;
    v[0].streamed = (readings & RD_FLUX_STREAMED) != 0;
    v[0].cls = h.cls.data();
    v[0].bnd = c.bnd.data();
    v[0].nb = (int64_t)c.bnd.size();
    PatchPlan p;
    const bool use = choose_plan(&c, v, p);
    printf("plan %d %d %d %d %zu %zu %.3f %.3f\n", use ? 1 : 0, p.K, p.rows, p.inner_rows, p.patches.size(),
           p.inner.size(), p.K ? block_us(&c, p) : 0.0, tile_us(&c));
    for (int K = 6; K >= 2; K--) {
      PatchPlan o;
      const bool cut = p.K && make_patch_plan(v, K, p.rows, p.inner_rows, o);
      printf("%d %.3f\n", K, cut ? block_us(&c, o) : 0.0);
    }
  }
  return 0;
}
