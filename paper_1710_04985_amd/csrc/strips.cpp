// Host side of the strip schedule: the grid behind a set of offsets, and the
// shape of the strips.
#include "strip_grid.hpp"

#include <algorithm>
#include <cstring>

namespace sptrsv {
namespace {

struct Off {
  int a, b, c;   // the entry lies a, b, c grid steps back (lexicographically positive in c, b, a)
};

// Strides and entry steps from the distinct offsets.
bool read_strides(const std::vector<int>& d, int n, int attempt, StripGrid& g,
                  std::vector<Off>& offs) {
  offs.clear();
  g.sy = g.sz = std::max(1, n);
  if (d.empty() || (d.size() == 1 && d[0] == 1)) {      // independent rows, or one chain
    if (attempt) return false;
    g.nx = n;
    g.ny = g.nz = 1;
    if (!d.empty()) offs.push_back({1, 0, 0});
    return true;
  }
  size_t at = d[0] == 1 ? 1 : 0;
  // the entries one line back: a run of at most three consecutive offsets
  size_t end = at + 1;
  while (end < d.size() && d[end] == d[end - 1] + 1) ++end;
  const size_t m = end - at;
  if (m > 3 || (attempt && m != 2)) return false;
  const int sy = d[at + (m == 3 ? 1 : m == 2 ? attempt : 0)];
  if (sy < 2) return false;
  int sz = 0;
  if (end < d.size()) {
    // the entries one plane back, centred on the plane stride
    sz = d[end + (d.size() - end) / 2];
    if (sz % sy || sz < 2 * sy) return false;
  }
  for (int v : d) {
    if (v == 1) {
      offs.push_back({1, 0, 0});
    } else if (v >= sy - 1 && v <= sy + 1) {
      offs.push_back({v - sy, 1, 0});
    } else {
      bool ok = false;
      for (int b = -1; b <= 1 && !ok && sz; ++b)
        for (int a = -1; a <= 1 && !ok; ++a)
          if (static_cast<int64_t>(sz) + static_cast<int64_t>(b) * sy + a == v) {
            offs.push_back({a, b, 1});
            ok = true;
          }
      if (!ok) return false;
    }
  }
  g.sy = sy;
  g.nx = sy;
  if (sz) {
    g.sz = sz;
    g.ny = sz / sy;
    g.nz = (n + sz - 1) / sz;
  } else {
    g.ny = (n + sy - 1) / sy;
    g.sz = sy * g.ny;
    g.nz = 1;
  }
  return true;
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Fills in the shape's tables (ghost lines, published lanes, farthest steps);
// false if they do not fit.
bool shape_tables(const std::vector<Off>& offs, StripGrid& g) {
  const int TU = 1 << g.lu, TV = 1 << g.lv;
  g.gu = g.gv = 0;
  g.dmax = 1;
  struct Back {
    int u, v;
  };
  std::vector<Back> back;
  for (const Off& o : offs) {
    const int c1 = o.a + g.al * o.b + g.be * o.c, c2 = o.b + g.ga * o.c, c3 = o.c;
    const int u = g.axis == 0 ? c2 : c1, v = g.axis == 2 ? c2 : c3;
    g.gu = std::max(g.gu, u);
    g.gv = std::max(g.gv, v);
    g.dmax = std::max(g.dmax, c1 + c2 + c3);
    back.push_back({u, v});
  }
  if (g.dmax > kStripMaxBack || (TU + g.gu) * (TV + g.gv) > 255) return false;
  std::memset(g.ghost, 255, sizeof(g.ghost));
  std::memset(g.pub, -1, sizeof(g.pub));
  std::memset(g.gcol, 0, sizeof(g.gcol));
  std::vector<char> need((TU + g.gu) * (TV + g.gv), 0);
  for (int v = 0; v < TV; ++v)
    for (int u = 0; u < TU; ++u)
      for (const Back& k : back)
        if (u < k.u || v < k.v) need[(u - k.u + g.gu) + (v - k.v + g.gv) * (TU + g.gu)] = 1;
  g.nghost = 0;
  for (size_t q = 0; q < need.size(); ++q)
    if (need[q]) {
      if (g.nghost == kMaxGhosts) return false;
      g.gcol[g.nghost] = static_cast<unsigned char>(q);
      g.ghost[q] = static_cast<unsigned char>(g.nghost++);
    }
  g.npub = 0;
  for (int l = 0; l < TU * TV; ++l)
    if ((l & (TU - 1)) >= TU - g.gu || (l >> g.lu) >= TV - g.gv) g.pub[l] = static_cast<signed char>(g.npub++);
  return true;
}

}  // namespace

bool strip_infer(const std::vector<int>& offsets, int n, bool upper, int attempt, StripGrid* out) {
  StripGrid g;
  std::vector<Off> offs;
  if (offsets.size() > kStripMaxOffsets || n < 1 || n >= (1 << 30)) return false;
  if (!read_strides(offsets, n, attempt, g, offs)) return false;
  if (static_cast<int64_t>(g.sy) * g.ny > (1ll << 30)) return false;
  g.n = n;
  g.upper = upper ? 1 : 0;
  for (const Off& o : offs) {
    if (o.c == 0 && o.b == 1) g.al = std::max(g.al, -o.a);
    if (o.c == 1) g.ga = std::max(g.ga, -o.b);
  }
  // every entry lies at least one level below its row
  for (const Off& o : offs)
    if (o.c == 0 && o.b == 0) g.wx = 1;
  for (const Off& o : offs)
    if (o.c == 0 && o.b == 1) g.wy = std::max(g.wy, 1 - g.wx * o.a);
  for (const Off& o : offs)
    if (o.c == 1) g.wz = std::max(g.wz, 1 - g.wx * o.a - g.wy * o.b);
  for (const Off& o : offs)
    if (o.c == 1) g.be = std::max(g.be, -(o.a + g.al * o.b));
  const int64_t ext[3] = {g.nx + static_cast<int64_t>(g.al) * (g.ny - 1) +
                              static_cast<int64_t>(g.be) * (g.nz - 1),
                          g.ny + static_cast<int64_t>(g.ga) * (g.nz - 1), g.nz};
  if (ext[0] > (1 << 30) || ext[1] > (1 << 30)) return false;
  // Shape: what differs is the chain of steps, and the work on lanes without a
  // row, counted here as steps of all strips over the wavefronts that share
  // them.  A line is walked step by step, and a lane starts one step after its
  // neighbour whether it needs it or not, so the chain has the steps of a line
  // and those of a strip's lanes; lines of other strips add theirs, and a hop,
  // worth about ten steps, per strip, only in a direction in which rows depend
  // on one another.  So a direction without dependencies, such as the lines of
  // a pattern with entries one plane back only, belongs across the lanes, not
  // along the walk.  (With dependencies in every direction all shapes have the
  // same chain, one step per level, but for the hops.)  Walking along x (axis
  // 0) reads b and writes x in order, so the others have to gain a quarter.
  StripGrid best;
  double best_cost = 0;
  bool found = false;
  for (int axis = 0; axis < 3; ++axis) {
    if ((axis == 1 && g.ny == 1) || (axis == 2 && g.nz == 1)) continue;
    const int64_t eu = axis == 0 ? ext[1] : ext[0], ev = axis == 2 ? ext[1] : ext[2];
    for (int lu = 0; lu <= 6; ++lu) {
      g.axis = axis;
      g.lu = lu;
      g.lv = 6 - lu;
      if (ev == 1 && g.lv > 0) continue;
      const int64_t nbu = ceil_div(eu, 1 << g.lu), nbv = ceil_div(ev, 1 << g.lv);
      if (nbu * nbv > static_cast<int64_t>(n) / 16 + 64 || !shape_tables(offs, g)) continue;
      const int64_t len = axis == 0 ? g.nx : axis == 1 ? g.ny : g.nz;
      const double steps = static_cast<double>(nbu * nbv) *
                           static_cast<double>(len + std::min<int64_t>(eu, 1 << g.lu) +
                                               std::min<int64_t>(ev, 1 << g.lv) - 2 + g.dmax);
      const int64_t lanes_u = g.gu ? eu : std::min<int64_t>(eu, 1 << g.lu),
                    lanes_v = g.gv ? ev : std::min<int64_t>(ev, 1 << g.lv);
      g.chain = static_cast<double>((axis == 0 ? ext[0] : axis == 1 ? ext[1] : ext[2]) + lanes_u +
                                    lanes_v) +
                10.0 * static_cast<double>((g.gu ? nbu - 1 : 0) + (g.gv ? nbv - 1 : 0));
      g.work = steps;
      double cost = g.chain + steps / 512;
      if (axis != 0) cost *= 1.25;
      g.nbu = static_cast<int>(nbu);
      g.nbv = static_cast<int>(nbv);
      if (!found || cost < best_cost) {
        found = true;
        best_cost = cost;
        best = g;
      }
    }
  }
  if (!found) return false;
  best.stride = best.axis == 0   ? 1
                : best.axis == 1 ? best.sy - best.al
                                 : best.sz - best.ga * best.sy + best.al * best.ga - best.be;
  if (upper) best.stride = -best.stride;
  *out = best;
  return true;
}

SolveCost strip_cost(const std::vector<StripGrid>& grids, int max_len, int vb) {
  SolveCost c;
  for (const StripGrid& g : grids) {
    if (g.n == 0) continue;
    c.chain = std::max(c.chain, g.chain);
    c.strips += static_cast<double>(g.nbu) * g.nbv;
    c.work += g.work;
  }
  const int slots = max_len > 4 ? 15 : std::max(2, max_len);
  c.words = (slots + 1) * (vb / 4) + (slots + 1) / 2;
  return c;
}

// Strips: 10 us of two launches (12.4 at least, call after call); 0.088 us a step
// of the chain (0.083 to 0.1
// measured); and the most of 0.0135 us a task, whose tickets are claimed one
// after another (4000 systems of 8x8, 1 / 8 columns: 64 / 385 us), 3500 steps of
// all tasks in a us (256 systems of 144x144, 1 / 8 columns: 88 / 463), and the
// records' bytes at 5 TB/s (columns find them in the cache: 100^3 27-point, 1 / 4
// columns: 245 / 254).
double strip_time(const SolveCost& c, int nrhs) {
  const double tasks = std::max(
      {0.0135 * c.strips * nrhs, c.work * nrhs / 3500, c.work * c.words * 256 / 5e6});
  return std::max(12.4, 10 + 0.088 * c.chain + tasks);
}

// Row by row: a hop per level, 0.7 us (rows of several lanes 1.2; several
// columns 0.8 and 1.6; the block schedule 0.35), and the rows' bytes where
// levels are wide.  Measured, us, strips / row-wise, with what the two
// functions give in brackets:
//   128^3 7-point, 382 levels                       99 / 373  (89 / 404)
//   128^2 5-point, half of the entries, 53 levels   33 / 52   (34 / 50)
//   128^2 5-point, a fifth of the entries, 10       33 / 19   (34 / 19)
//   512^2 5-point, a third of the entries, 22      107 / 44   (108 / 34)
//   offset 16,384 only on 2 M rows, 128 levels      32 / 121  (45 / 164)
//   16,384 rows in 64 chains, 256 levels          1369 / 177  (1458 / 192)
//   20,000 independent rows                       1694 / 16   (1777 / 13)
//   1000 systems of 16x16, 31 levels                33 / 46   (26 / 45)
//   the same, eight columns                        113 / 83   (121 / 88)
//   5 rows in a chain, against the block schedule 12.3 / 10.8 (12.4 / 10.8)
double row_time(int64_t n, int64_t noff, int nlev, int max_len, bool block, int nrhs) {
  if (nrhs > 1)
    return 24 + (max_len > 4 ? 1.6 : 0.8) * nlev + 1.9e-5 * static_cast<double>(n) * nrhs;
  if (block) return std::max(10.8, 6.5 + 0.35 * nlev);   // one launch
  return 12 + (max_len > 4 ? 1.2 : 0.7) * nlev + 1.5e-5 * static_cast<double>(n + noff);
}

}  // namespace sptrsv
