// Host side of the tiled schedule: the grid behind a set of offsets, and the
// tile shape.
#include "tiles.hpp"

#include <algorithm>
#include <set>

namespace sptrsv {
namespace {

struct Off {
  int a, b, c;   // the entry lies a, b, c grid steps back (lexicographically positive in c, b, a)
};

// Strides and entry steps from the distinct offsets.
bool read_strides(const std::vector<int>& d, int n, int attempt, TileGrid& g,
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

}  // namespace

bool tile_infer(const std::vector<int>& offsets, int n, bool upper, int attempt, TileGrid* out,
                int* ext) {
  TileGrid g;
  std::vector<Off> offs;
  if (offsets.size() > kTileMaxOffsets || n < 1 || n >= (1 << 30)) return false;
  if (!read_strides(offsets, n, attempt, g, offs)) return false;
  // sy * ny may exceed n only by the last, partial line
  if (static_cast<int64_t>(g.sy) * g.ny > (1ll << 30)) return false;
  g.n = n;
  g.upper = upper ? 1 : 0;
  for (const Off& o : offs) {
    if (o.c == 0 && o.b == 1) g.al = std::max(g.al, -o.a);
    if (o.c == 1) g.ga = std::max(g.ga, -o.b);
  }
  for (const Off& o : offs)
    if (o.c == 1) g.be = std::max(g.be, -(o.a + g.al * o.b));
  g.be = std::max(g.be, g.al * g.ga);
  const int64_t e1 = g.nx + static_cast<int64_t>(g.al) * (g.ny - 1) +
                     static_cast<int64_t>(g.be) * (g.nz - 1);
  const int64_t e2 = g.ny + static_cast<int64_t>(g.ga) * (g.nz - 1);
  if (e1 > (1 << 30) || e2 > (1 << 30)) return false;
  // Tile shape: the chain crosses about e1/tx + e2/ty + e3/tz tiles, each
  // costing one hop and tx + ty + tz - 2 steps inside the tile; a step costs
  // about a tenth of a hop.  Boxes that reach past the grid cost their share.
  double best = 0;
  bool found = false;
  for (int lx = 0; lx <= 6; ++lx)
    for (int ly = 0; lx + ly <= 6; ++ly) {
      const int lz = 6 - lx - ly;
      if ((g.nz == 1 && lz > 0) || (g.ny == 1 && g.nz == 1 && ly > 0)) continue;
      const int tx = 1 << lx, ty = 1 << ly, tz = 1 << lz;
      const double depth = static_cast<double>(ceil_div(e1, tx) + ceil_div(e2, ty) +
                                               ceil_div(g.nz, tz) - 2);
      const double step = 1.0 + 0.1 * (tx + ty + tz - 2);
      const double fill = static_cast<double>(ceil_div(g.nx, tx) * tx) / g.nx *
                          (static_cast<double>(ceil_div(g.ny, ty) * ty) / g.ny) *
                          (static_cast<double>(ceil_div(g.nz, tz) * tz) / g.nz);
      const double cost = depth * step * (0.5 + 0.5 * fill);
      if (!found || cost < best) {
        found = true;
        best = cost;
        g.lx = lx;
        g.ly = ly;
        g.lz = lz;
      }
    }
  const int tx = 1 << g.lx, ty = 1 << g.ly, tz = 1 << g.lz;
  const int k = g.be - g.al * g.ga;
  const int64_t nbx = (g.nx - 1 + static_cast<int64_t>(g.al) * (ty - 1) +
                       static_cast<int64_t>(k) * (tz - 1) + tx - 1) / tx + 1;
  const int64_t nby = (g.ny - 1 + static_cast<int64_t>(g.ga) * (tz - 1) + ty - 1) / ty + 1;
  const int64_t nbz = ceil_div(g.nz, tz);
  if (nbx * nby * nbz > static_cast<int64_t>(n) / 4 + 4096) return false;
  g.nbx = static_cast<int>(nbx);
  g.nby = static_cast<int>(nby);
  g.nbz = static_cast<int>(nbz);
  // values a full tile needs from outside (tiles at the edge need fewer)
  std::set<std::vector<int>> need;
  for (int w = 0; w < tz; ++w)
    for (int v = 0; v < ty; ++v)
      for (int u = 0; u < tx; ++u)
        for (const Off& o : offs) {
          const int c1 = u - (o.a + g.al * o.b + g.be * o.c), c2 = v - (o.b + g.ga * o.c),
                    c3 = w - o.c;
          if (c1 < 0 || c2 < 0 || c3 < 0) need.insert({c1, c2, c3});
        }
  *ext = static_cast<int>(need.size());
  *out = g;
  return *ext <= kTileMaxExt;
}

}  // namespace sptrsv
