// Host-only check (no GPU): no exception leaves the planning of block passes or
// the tiles of a context when host memory runs out, at any allocation of more
// than 256 bytes (an error text still finds room).  Built by
// tests/test_no_memory_cpu.py; the kernel launchers are stubs.
//
// stdout: per call "name allocations A failed F" (F: calls that reported it)
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>

static std::atomic<long> g_left{-1}, g_count{0};  // -1: not armed

void *operator new(std::size_t n) {
  if (g_left >= 0 && n > 256) {
    g_count++;
    if (g_left-- <= 0) {
      g_left = 0;
      throw std::bad_alloc();
    }
  }
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

#define main tiles_main
#include "tiles_harness.cpp"
#undef main

// (the device's allocator: the host allocations to be tried are done by then)
static void *refuse(size_t, void *) {
  g_left = -1;
  return nullptr;
}
static void nothing(void *, void *) {}

static void body(lbm_ctx &c, std::vector<uint8_t> &mask) {
  lbm_plate pl{};
  pl.nx = 700;
  pl.ny = 400;
  mask.assign((size_t)pl.nx * pl.ny, 1);
  for (int j = 100; j < 140; j++)
    for (int i = 90; i < 150; i++) mask[(size_t)j * pl.nx + i] = 0;
  pl.mask = mask.data();
  c.ph.resize(1);
  c.pd.resize(1);
  PlateHost &h = c.ph[0];
  h.nx = pl.nx;
  h.ny = pl.ny;
  h.pitch = 704;
  std::string why;
  if (!classify(pl, h, why)) std::exit(3);
  c.n_body = h.body;
  for (int j = 0; j < pl.ny; j++)
    for (int i = 0; i < pl.nx; i++) {
      const uint8_t cl = h.cls[(size_t)j * pl.nx + i];
      if (cl & CL_B) {
        BndNode b{};
        b.i = i;
        b.j = j;
        b.node = (int64_t)j * h.pitch + i;
        c.bnd.push_back(b);
      } else if (cl & CL_S) {
        SecNode s{};
        s.i = i;
        s.j = j;
        s.node = (int64_t)j * h.pitch + i;
        c.sec.push_back(s);
      }
    }
  h.b1 = (int64_t)c.bnd.size();
  c.have_alloc = true;
  c.alloc.alloc = refuse;
  c.alloc.free = nothing;
}

template <class F>
static void sweep(const char *name, F &&call) {
  long total = 0, failed = 0;
  for (long k = -1; k < 0 || k < total; k += k < 64 ? 1 : 1 + total / 96) {
    lbm_ctx c;
    std::vector<uint8_t> mask;
    body(c, mask);
    g_count = 0;
    g_left = k < 0 ? 1000000000 : k;
    const bool ok = call(c);
    g_left = -1;
    if (k < 0) total = g_count;
    failed += ok ? 0 : 1;
  }
  printf("%s allocations %ld failed %ld\n", name, total, failed);
  fflush(stdout);
}

int main() {
  sweep("plan_blocks", [](lbm_ctx &c) { return plan_blocks(&c); });
  sweep("new_tiles", [](lbm_ctx &c) { return new_tiles(&c) == LBM_OK; });
  sweep("new_tiles of block passes", [](lbm_ctx &c) {
    c.block = true;
    return new_tiles(&c) == LBM_OK;
  });
  return 0;
}
