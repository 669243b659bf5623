// lbm_patches.h -- the patches of the block pass (host code, header only).
//
// Cuts a plate into rectangles and finds, for each, the smallest rectangle of
// nodes around it that K steps of its nodes depend on.
#pragma once

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <thread>
#include <utility>
#include <vector>

#include "lbm_types.h"

namespace lbm {

struct PatchPlate {
  int index = 0;                 // plate
  int nx = 0, ny = 0;
  bool px = false, py = false;   // periodic axes
  bool streamed = false;         // reading R2
  const uint8_t *cls = nullptr;  // dense nx * ny class bytes
  const BndNode *bnd = nullptr;  // the plate's boundary records, row-major
  int64_t nb = 0, b0 = 0;        // their number, index of the first one
};

// What the patches of a plan are cut for: K steps, rows per wave of those with
// boundary nodes, rows of those without (`inner`) at most.
struct PatchPlan {
  int K = 0, rows = 0, inner_rows = 0;
  std::vector<Patch> patches, inner;
  std::vector<PTask> tasks;
  std::vector<PGrad> grads;
};

class PatchCutter {
 public:
  // made, most: patches made so far, of all plates; a cut that would make more
  // than `most` fails
  PatchCutter(const PatchPlate &p, int K, int rows, int inner, std::atomic<int64_t> *made = nullptr,
              int64_t most = INT64_MAX)
      : p_(p), K_(K), hb_(rows * (kBlockThreads / 64 - 1)), hi_(inner),
        ring_(3 * K + 4), made_(made), most_(most) {
    row0_.assign((size_t)p.ny + 1, 0);
    for (int64_t b = 0; b < p.nb; b++) row0_[(size_t)p.bnd[b].j + 1]++;
    for (int j = 0; j < p.ny; j++) row0_[(size_t)j + 1] += row0_[(size_t)j];
  }

  // Rectangles of the plate to cut, [x0, x1) x [y0, y1), and the largest pieces
  // to cut them into (w x h nodes; the outermost columns of a piece at a bounded
  // x edge may be wider: we).
  struct Band {
    int x0, x1, y0, y1;
    int w, we;
  };
  // Boundary nodes reach 2 K + 2 nodes along the boundary and K + 3 away from it;
  // a patch without any depends on K nodes all around.
  std::vector<Band> bands() const {
    std::vector<Band> v;
    const int W = kBlockCols, along = 2 * K_ + 2, off = K_ + 3;
    const int we = std::max(1, W - along);      // piece of a band along a y edge
    const int he = std::max(1, hb_ - off);      // its rows
    const int ws = std::max(1, W / 2 - off);    // columns along an x edge, in tall patches
    const int hs = std::max(1, 2 * hb_ - 2 * along);  // their rows
    auto rows = [&](int x0, int x1, int a, int b, int h, int w, int wedge) {
      const int n = (b - a + h - 1) / h;
      for (int i = 0; i < n; i++)
        v.push_back({x0, x1, a + (int)((int64_t)(b - a) * i / n), a + (int)((int64_t)(b - a) * (i + 1) / n), w, wedge});
    };
    int y0 = 0, y1 = p_.ny;
    if (!p_.py) {
      const int wedge = p_.px ? 0 : W - along;
      if (p_.ny <= 2 * he) {
        rows(0, p_.nx, 0, p_.ny, p_.ny <= hb_ ? p_.ny : he, we, wedge);
        return v;
      }
      y0 = he;
      y1 = p_.ny - he;
      rows(0, p_.nx, 0, y0, he, we, wedge);
      rows(0, p_.nx, y1, p_.ny, he, we, wedge);
    }
    int x0 = 0, x1 = p_.nx;
    if (!p_.px) {
      if (p_.nx <= 2 * ws) {
        rows(0, p_.nx, y0, y1, hs, ws, 0);
        return v;
      }
      x0 = ws;
      x1 = p_.nx - ws;
      rows(0, x0, y0, y1, hs, ws, 0);
      rows(x1, p_.nx, y0, y1, hs, ws, 0);
    }
    rows(x0, x1, y0, y1, std::max(1, hi_ - 2 * K_), std::max(1, W - 2 * K_), 0);
    return v;
  }

  // The patches of one band; false if some node's dependences do not fit, or past
  // `most`.
  bool cut(const Band &b, PatchPlan &out) {
    bool ok = true;
    auto even = [&](int x0, int x1, int w) {
      const int n = (x1 - x0 + w - 1) / w;
      for (int i = 0; i < n && ok; i++)
        ok = place(x0 + (int)((int64_t)(x1 - x0) * i / n), x0 + (int)((int64_t)(x1 - x0) * (i + 1) / n),
                   b.y0, b.y1, out);
    };
    const int nx = b.x1 - b.x0;
    if (b.we > 0 && nx <= kBlockCols) {
      even(b.x0, b.x1, nx);
    } else if (b.we > 0 && nx > 2 * b.we) {
      even(b.x0, b.x0 + b.we, b.we);
      even(b.x0 + b.we, b.x1 - b.we, b.w);
      even(b.x1 - b.we, b.x1, b.we);
    } else {
      even(b.x0, b.x1, b.w);
    }
    return ok;
  }

  // The dependence region of K steps of the nodes [x0, x1) x [y0, y1): the
  // smallest rectangle [ex, ex + ew) x [ey, ey + eh) (not wrapped) that holds
  // every node whose state at t they depend on; nb: its boundary nodes (0:
  // none of the K steps touches one).  False: no node of it is in the body.
  //
  // Rules, from the method.  Populations of t + j (F) need at an interior
  // node those of t + j - 1 at the node and its four neighbours, and at a
  // neighbour that is a boundary node also its reset field at t + j; at a
  // boundary node u of t + j on its finite-difference stencil (and, under reading
  // R2, the neighbours' F of t + j - 1).  u, du/dt of
  // t + j (U) need those of t + j - 1 at the node and, at an interior node,
  // the neighbours' fields of t + j - 1, at a boundary node u of t + j - 1 on
  // the stencils of the node and its body neighbours.
  bool region(int x0, int x1, int y0, int y1, int &ex, int &ey, int &ew, int &eh, int &nb) {
    if (!any_boundary(x0 - K_, x1 + K_, y0 - K_, y1 + K_)) {
      // (the body begins and ends at boundary nodes)
      if (!(p_.cls[(size_t)y0 * p_.nx + x0] & CL_IN)) return false;
      ex = x0 - K_;
      ey = y0 - K_;
      ew = x1 - x0 + 2 * K_;
      eh = y1 - y0 + 2 * K_;
      nb = 0;
      return true;
    }
    lx_ = x0 - ring_;
    ly_ = y0 - ring_;
    gw_ = x1 - x0 + 2 * ring_;
    gh_ = y1 - y0 + 2 * ring_;
    load_classes();
    lf_.assign(c_.size(), -1);
    lu_.assign(c_.size(), -1);
    queue_.resize((size_t)K_ + 1);
    for (auto &q : queue_) q.clear();
    minx_ = miny_ = INT32_MAX;
    maxx_ = maxy_ = INT32_MIN;
    // the rectangle's own nodes; what a node not at its border and not next to
    // the boundary depends on is among them
    for (int j = y0; j < y1; j++)
      for (int i = x0; i < x1; i++) {
        const int k = id(i, j);
        const uint8_t c = c_[(size_t)k];
        if (!(c & CL_IN)) continue;
        extend(i, j);
        lf_[(size_t)k] = lu_[(size_t)k] = (int8_t)K_;
        if ((c & (CL_B | CL_S)) || j == y0 || j == y1 - 1 || i == x0 || i == x1 - 1) {
          queue_[(size_t)K_].push_back({k, false});
          queue_[(size_t)K_].push_back({k, true});
        }
      }
    if (maxx_ < minx_) return false;
    for (int l = K_; l >= 0; l--)
      for (size_t q = 0; q < queue_[(size_t)l].size(); q++) {  // (grows while it is walked)
        const Item it = queue_[(size_t)l][q];
        if (it.u) {
          if (lu_[(size_t)it.k] == l) expand_u(it.k, l);
        } else if (lf_[(size_t)it.k] == l) {
          expand_f(it.k, l);
        }
      }
    ex = minx_;
    ey = miny_;
    ew = maxx_ - minx_ + 1;
    eh = maxy_ - miny_ + 1;
    nb = 0;
    for (int j = ey; j < ey + eh; j++)
      for (int i = ex; i < ex + ew; i++) nb += (at(i, j) & CL_B) ? 1 : 0;
    return true;
  }

 private:
  struct Item {
    int k;
    bool u;
  };
  PatchPlate p_;
  int K_, hb_, hi_, ring_;
  std::atomic<int64_t> *made_;
  int64_t most_;
  std::vector<int64_t> row0_;
  int lx_ = 0, ly_ = 0, gw_ = 0, gh_ = 0;
  std::vector<uint8_t> c_;
  std::vector<int8_t> lf_, lu_;  // largest level at which a node's F / U is needed (-1: not)
  std::vector<std::vector<Item>> queue_;
  std::vector<std::pair<int, int>> g_;  // gradient nodes of the patch being placed
  std::vector<int> gi_;                 // their index by node (-1: none)
  int minx_ = 0, miny_ = 0, maxx_ = 0, maxy_ = 0;

  void load_classes() {
    c_.assign((size_t)gw_ * gh_, 0);
    for (int j = 0; j < gh_; j++) {
      int y = ly_ + j;
      if (p_.py)
        y = ((y % p_.ny) + p_.ny) % p_.ny;
      else if (y < 0 || y >= p_.ny)
        continue;
      const uint8_t *src = p_.cls + (size_t)y * p_.nx;
      uint8_t *dst = c_.data() + (size_t)j * gw_;
      if (p_.px) {
        int x = ((lx_ % p_.nx) + p_.nx) % p_.nx;
        for (int i = 0; i < gw_; i++) {
          dst[i] = src[x];
          if (++x == p_.nx) x = 0;
        }
      } else {
        const int a = std::max(0, lx_), b = std::min(p_.nx, lx_ + gw_);
        if (b > a) std::copy(src + a, src + b, dst + (a - lx_));
      }
    }
  }
  // Some boundary node in [x0, x1) x [y0, y1) (not wrapped)?
  bool any_boundary(int x0, int x1, int y0, int y1) const {
    for (int j = y0; j < y1; j++) {
      int y = j;
      if (p_.py)
        y = ((j % p_.ny) + p_.ny) % p_.ny;
      else if (j < 0 || j >= p_.ny)
        continue;
      const BndNode *r0 = p_.bnd + row0_[(size_t)y], *r1 = p_.bnd + row0_[(size_t)y + 1];
      if (r0 == r1) continue;
      // (on a periodic axis also the parts past either end; a plate narrower than
      // that is one with some anywhere)
      if (p_.px && x1 - x0 >= p_.nx) return true;
      for (int sh = p_.px ? -1 : 0; sh <= (p_.px ? 1 : 0); sh++) {
        const int a = x0 + sh * p_.nx, b = x1 + sh * p_.nx;
        const BndNode *r = std::lower_bound(r0, r1, a, [](const BndNode &n, int v) { return n.i < v; });
        if (r != r1 && r->i < b) return true;
      }
    }
    return false;
  }
  int id(int i, int j) const { return (j - ly_) * gw_ + (i - lx_); }
  bool inside(int i, int j) const { return i >= lx_ && i < lx_ + gw_ && j >= ly_ && j < ly_ + gh_; }
  uint8_t at(int i, int j) const { return inside(i, j) ? c_[(size_t)id(i, j)] : 0; }

  // Stencil code of the finite difference along axis ax.
  int code(int i, int j, int ax) const {
    const uint8_t c0 = at(i, j), bp = ax == 0 ? NB_E : NB_N, bm = ax == 0 ? NB_W : NB_S;
    const int di = ax == 0, dj = ax != 0;
    if ((c0 & bp) && (c0 & bm)) return FD_CENTRAL;
    if (c0 & bp) return (at(i + di, j + dj) & bp) ? FD_FWD3 : FD_FWD2;
    if (c0 & bm) return (at(i - di, j - dj) & bm) ? FD_BWD3 : FD_BWD2;
    return FD_NONE;
  }

  void extend(int i, int j) {
    minx_ = std::min(minx_, i);
    maxx_ = std::max(maxx_, i);
    miny_ = std::min(miny_, j);
    maxy_ = std::max(maxy_, j);
  }
  void need_f(int i, int j, int l) {
    if (!(at(i, j) & CL_IN)) return;
    int8_t &v = lf_[(size_t)id(i, j)];
    if (v >= l) return;
    if (v < 0) extend(i, j);
    v = (int8_t)l;
    queue_[(size_t)l].push_back({id(i, j), false});
  }
  void need_u(int i, int j, int l) {
    if (!(at(i, j) & CL_IN)) return;
    int8_t &v = lu_[(size_t)id(i, j)];
    if (v >= l) return;
    if (v < 0) extend(i, j);
    v = (int8_t)l;
    queue_[(size_t)l].push_back({id(i, j), true});
  }
  void need_stencil(int i, int j, int l) {
    need_u(i, j, l);
    for (int ax = 0; ax < 2; ax++) {
      const int di = ax == 0, dj = ax != 0;
      switch (code(i, j, ax)) {
        case FD_CENTRAL: need_u(i + di, j + dj, l); need_u(i - di, j - dj, l); break;
        case FD_FWD3: need_u(i + 2 * di, j + 2 * dj, l);  // fall through
        case FD_FWD2: need_u(i + di, j + dj, l); break;
        case FD_BWD3: need_u(i - 2 * di, j - 2 * dj, l);  // fall through
        case FD_BWD2: need_u(i - di, j - dj, l); break;
        default: break;
      }
    }
  }
  template <class F>
  void neighbours(int i, int j, F &&fn) {
    fn(i + 1, j);
    fn(i, j + 1);
    fn(i - 1, j);
    fn(i, j - 1);
  }
  void expand_f(int k, int l) {
    const int i = lx_ + k % gw_, j = ly_ + k / gw_;
    if (l == 0) return;
    if (c_[(size_t)k] & CL_B) {
      need_stencil(i, j, l);
      if (p_.streamed) neighbours(i, j, [&](int a, int b) { need_f(a, b, l - 1); });
      return;
    }
    need_f(i, j, l - 1);
    neighbours(i, j, [&](int a, int b) {
      need_f(a, b, l - 1);
      if (at(a, b) & CL_B) need_f(a, b, l);
    });
  }
  void expand_u(int k, int l) {
    const int i = lx_ + k % gw_, j = ly_ + k / gw_;
    if (l == 0) return;
    need_u(i, j, l - 1);
    if (c_[(size_t)k] & CL_B) {
      need_stencil(i, j, l - 1);
      neighbours(i, j, [&](int a, int b) {
        if (at(a, b) & CL_IN) need_stencil(a, b, l - 1);
      });
    } else {
      neighbours(i, j, [&](int a, int b) { need_f(a, b, l - 1); });
    }
  }

  // The gradient nodes of the patch's boundary nodes: those first (in the
  // order of the tasks), then their other body neighbours within the patch.
  int gradients(const Patch &t) {
    g_.clear();
    gi_.assign(c_.size(), -1);
    for (int j = t.ey; j < t.ey + t.eh; j++)
      for (int i = t.ex; i < t.ex + t.ew; i++)
        if (at(i, j) & CL_B) {
          gi_[(size_t)id(i, j)] = (int)g_.size();
          g_.push_back({i, j});
        }
    const size_t nb = g_.size();
    for (size_t q = 0; q < nb; q++)
      neighbours(g_[q].first, g_[q].second, [&](int a, int b) {
        if (a < t.ex || a >= t.ex + t.ew || b < t.ey || b >= t.ey + t.eh || !(at(a, b) & CL_IN)) return;
        int &v = gi_[(size_t)id(a, b)];
        if (v >= 0) return;
        v = (int)g_.size();
        g_.push_back({a, b});
      });
    return (int)g_.size();
  }

  bool place(int x0, int x1, int y0, int y1, PatchPlan &out) {
    Patch t{};
    int nb = 0;
    if (!region(x0, x1, y0, y1, t.ex, t.ey, t.ew, t.eh, nb)) return true;  // nothing there
    const int w = x1 - x0, h = y1 - y0;
    // the shape that takes fewer pieces
    t.w = kBlockCols;
    int ox = t.ew - kBlockCols, oy = t.eh - (nb ? hb_ : hi_);
    if (nb && (ox > 0 || oy > 0)) {
      auto pieces = [](int n, int over) {  // of an axis whose excess is `over`
        return over <= 0 ? 1 : n - over >= 1 ? (n + n - over - 1) / (n - over) : 4 * n;
      };
      const int ox2 = t.ew - kBlockCols / 2, oy2 = t.eh - 2 * hb_;
      if (pieces(w, ox2) * pieces(h, oy2) < pieces(w, ox) * pieces(h, oy)) {
        t.w = kBlockCols / 2;
        ox = ox2;
        oy = oy2;
      }
    }
    if (ox > 0 || oy > 0 || nb > kBlockTasks || (nb && gradients(t) > kBlockGrads)) {
      // into as many equal parts as leave the excess out, along the axis in excess
      const bool sx = ox > 0 ? true : oy > 0 ? false : w >= h;
      const int n = sx ? w : h, over = sx ? ox : oy;
      if (n < 2) return false;
      const int keep = over > 0 ? n - over : n / 2;
      const int parts = keep >= 1 ? std::max(2, (n + keep - 1) / keep) : 2;
      bool ok = true;
      for (int i = 0; i < parts && ok; i++) {
        const int a = (int)((int64_t)n * i / parts), b = (int)((int64_t)n * (i + 1) / parts);
        if (a == b) continue;
        ok = sx ? place(x0 + a, x0 + b, y0, y1, out) : place(x0, x1, y0 + a, y0 + b, out);
      }
      return ok;
    }
    if (made_ && ++*made_ > most_) return false;
    t.plate = p_.index;
    // (the rectangle's body nodes are all in the patch)
    t.ox0 = std::max(0, x0 - t.ex);
    t.ox1 = std::min(t.ew, x1 - t.ex);
    t.oy0 = std::max(0, y0 - t.ey);
    t.oy1 = std::min(t.eh, y1 - t.ey);
    t.b0 = (int)out.tasks.size();
    t.g0 = (int)out.grads.size();
    for (int q = 0; q < (nb ? (int)g_.size() : 0); q++) {
      const int i = g_[(size_t)q].first, j = g_[(size_t)q].second;
      PGrad G{};
      G.l = (uint16_t)((j - t.ey) * t.w + (i - t.ex));
      G.code = (uint16_t)(code(i, j, 0) | (code(i, j, 1) << 3));
      G.task = q < nb ? (int16_t)q : (int16_t)-1;
      out.grads.push_back(G);
      if (q >= nb) continue;
      const int x = ((i % p_.nx) + p_.nx) % p_.nx, y = ((j % p_.ny) + p_.ny) % p_.ny;
      const BndNode *r0 = p_.bnd + row0_[(size_t)y], *r1 = p_.bnd + row0_[(size_t)y + 1];
      const BndNode *r = std::lower_bound(r0, r1, x, [](const BndNode &b, int v) { return b.i < v; });
      PTask T{};
      T.bnd = (int32_t)(p_.b0 + (r - p_.bnd));
      T.l = G.l;
      T.own = i >= x0 && i < x1 && j >= y0 && j < y1;
      T.g[0] = (int16_t)q;
      int d = 1;
      // (a neighbour past the patch: the node is one whose result is not needed)
      neighbours(i, j, [&](int a, int b) {
        const bool in = a >= t.ex && a < t.ex + t.ew && b >= t.ey && b < t.ey + t.eh;
        T.g[d++] = in ? (int16_t)gi_[(size_t)id(a, b)] : (int16_t)-1;
      });
      out.tasks.push_back(T);
    }
    t.b1 = (int)out.tasks.size();
    t.g1 = (int)out.grads.size();
    out.patches.push_back(t);
    return true;
  }
};

// The plan for K steps with `rows` rows per wave (patches without boundary
// nodes: `inner` rows at most) over all plates; false if some plate cannot be cut
// (a node's dependences exceed a patch) or takes more than `most` patches, which
// ends the cut there: a body too dense in boundary nodes for K steps would be cut
// into tens of thousands (a second and more of host work).  Bands are cut by
// several host threads; the result does not depend on their number.
inline bool make_patch_plan(const std::vector<PatchPlate> &plates, int K, int rows, int inner,
                            PatchPlan &plan, int64_t most = INT64_MAX) {
  struct Job {
    int plate;
    PatchCutter::Band band;
    PatchPlan out;
    bool ok = false;
  };
  std::vector<Job> jobs;
  int64_t nodes = 0, bounded = 0;
  for (size_t p = 0; p < plates.size(); p++) {
    PatchCutter c(plates[p], K, rows, inner);
    for (const auto &b : c.bands()) jobs.push_back(Job{(int)p, b, {}, false});
    nodes += (int64_t)plates[p].nx * plates[p].ny;
    bounded += plates[p].nb;
  }
  std::atomic<size_t> next{0};
  std::atomic<bool> failed{false};
  std::atomic<int64_t> made{0};
  auto work = [&]() {
    try {
      int have = -1;
      std::vector<PatchCutter> cutter;
      for (size_t i = next++; i < jobs.size() && !failed; i = next++) {
        if (have != jobs[i].plate) {
          cutter.clear();
          cutter.emplace_back(plates[(size_t)jobs[i].plate], K, rows, inner, &made, most);
          have = jobs[i].plate;
        }
        jobs[i].ok = cutter[0].cut(jobs[i].band, jobs[i].out);
        if (!jobs[i].ok) failed = true;
      }
    } catch (...) {
      failed = true;
    }
  };
  // (a thread costs about as much as cutting a quarter of a million nodes or half a
  // thousand boundary nodes)
  const size_t want = (size_t)std::min<int64_t>(
      std::min<int64_t>(16, (int64_t)std::thread::hardware_concurrency()), nodes / (1 << 18) + bounded / 512);
  std::vector<std::thread> pool;
  try {
    for (size_t i = 1; i < std::min(want, jobs.size()); i++) pool.emplace_back(work);
  } catch (...) {
    // fewer threads
  }
  work();
  for (auto &t : pool) t.join();
  if (failed) return false;
  plan.K = K;
  plan.rows = rows;
  plan.inner_rows = inner;
  plan.patches.clear();
  plan.inner.clear();
  plan.tasks.clear();
  plan.grads.clear();
  for (Job &j : jobs) {
    const int tb = (int)plan.tasks.size(), gb = (int)plan.grads.size();
    for (Patch t : j.out.patches) {
      t.b0 += tb;
      t.b1 += tb;
      t.g0 += gb;
      t.g1 += gb;
      (t.b1 > t.b0 ? plan.patches : plan.inner).push_back(t);
    }
    plan.tasks.insert(plan.tasks.end(), j.out.tasks.begin(), j.out.tasks.end());
    plan.grads.insert(plan.grads.end(), j.out.grads.begin(), j.out.grads.end());
  }
  return true;
}

}  // namespace lbm
