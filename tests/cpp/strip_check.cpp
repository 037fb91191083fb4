// CPU model of the strip form's geometry and LDS ring, for patterns given as
// CSR: walks every strip as the solve kernel does, with row numbers in place
// of values, and checks that every entry reads its own dependency.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <set>
#include <vector>

#include "strip_grid.hpp"

using namespace sptrsv;

namespace {

// `lead`: how many steps ahead of the solver the ghost values are brought in
int walk(const StripGrid& g, const int* rp, const int* ci, int lead) {
  const int TU = 1 << g.lu, TV = 1 << g.lv;
  struct Strip {
    int bu, bv, first, end;
  };
  std::vector<Strip> strips;
  for (int bv = 0; bv < g.nbv; ++bv)
    for (int bu = 0; bu < g.nbu; ++bu) {
      int first = INT32_MAX, end = INT32_MIN;
      for (int l = 0; l < 64; ++l) {
        const int u = bu * TU + (l & (TU - 1)), v = bv * TV + (l >> g.lu);
        int lo, hi;
        strip_line(g, u, v, &lo, &hi);
        if (hi > lo) {
          first = std::min(first, lo + u + v);
          end = std::max(end, hi + u + v);
        }
      }
      if (end > first) strips.push_back({bu, bv, first - g.dmax, end});
    }
  std::stable_sort(strips.begin(), strips.end(),
                   [](const Strip& a, const Strip& b) { return a.bu + a.bv < b.bu + b.bv; });
  std::vector<char> solved(g.n, 0);
  for (const Strip& s : strips) {
    std::vector<int> ring(kRingSteps * kRingCols, -1);
    std::vector<int> lo(64), hi(64), glo(64, 0), ghi(64, 0), gu(64), gv(64);
    for (int l = 0; l < 64; ++l)
      strip_line(g, s.bu * TU + (l & (TU - 1)), s.bv * TV + (l >> g.lu), &lo[l], &hi[l]);
    for (int q = 0; q < g.nghost; ++q) {
      const int W = TU + g.gu;
      gu[q] = s.bu * TU + g.gcol[q] % W - g.gu;
      gv[q] = s.bv * TV + g.gcol[q] / W - g.gv;
      if (gu[q] < 0 || gv[q] < 0) continue;
      strip_line(g, gu[q], gv[q], &glo[q], &ghi[q]);
      if (ghi[q] > glo[q] && g.pub[(gu[q] & (TU - 1)) | ((gv[q] & (TV - 1)) << g.lu)] < 0) return 1;
    }
    int brought = 0;
    for (int step = 0; step < s.end - s.first; ++step) {
      for (; brought < step + lead; ++brought)
        for (int q = 0; q < g.nghost; ++q) {
          const int w = brought + s.first - gu[q] - gv[q];
          if (w < glo[q] || w >= ghi[q]) continue;
          const int r = strip_row(g, StripPoint{gu[q], gv[q], w});
          if (r < 0 || !solved[r]) return 2;          // from an earlier strip, and solved
          ring[(brought % kRingSteps) * kRingCols + 64 + q] = r;
        }
      std::vector<int> now(64, -1);
      for (int l = 0; l < 64; ++l) {
        const int u = s.bu * TU + (l & (TU - 1)), v = s.bv * TV + (l >> g.lu);
        const int w = step + s.first - u - v;
        if (w < lo[l] || w >= hi[l]) continue;
        const int r = strip_row(g, StripPoint{u, v, w});
        if (r < 0 || r != strip_row(g, StripPoint{u, v, lo[l]}) + (w - lo[l]) * g.stride) return 3;
        for (int e = rp[r]; e < rp[r + 1]; ++e) {
          if (ci[e] == r) continue;
          const StripPoint t = strip_point(g, ci[e]);
          const int back = step - (t.u + t.v + t.w - s.first);
          const int du = t.u - s.bu * TU, dv = t.v - s.bv * TV;
          if (back < 1 || back > g.dmax || du >= TU || dv >= TV || du < -g.gu || dv < -g.gv)
            return 4;                                 // the library keeps such a pattern row-wise
          int col = du >= 0 && dv >= 0 ? du | (dv << g.lu)
                                       : g.ghost[(du + g.gu) + (dv + g.gv) * (TU + g.gu)];
          if (du < 0 || dv < 0) {
            if (col >= kMaxGhosts) return 5;
            col += 64;
          }
          if (ring[((step - back) % kRingSteps) * kRingCols + col] != ci[e]) return 6;
        }
        now[l] = r;
      }
      for (int l = 0; l < 64; ++l)
        if (now[l] >= 0) {
          ring[(step % kRingSteps) * kRingCols + l] = now[l];
          if (solved[now[l]]) return 7;
          solved[now[l]] = 1;
        }
    }
  }
  for (char c : solved)
    if (!c) return 8;
  return 0;
}

bool infer(int n, const int* rp, const int* ci, int upper, int attempt, StripGrid* g) {
  std::set<int> d;
  for (int i = 0; i < n; ++i)
    for (int e = rp[i]; e < rp[i + 1]; ++e)
      if (ci[e] != i) d.insert(std::abs(ci[e] - i));
  return strip_infer(std::vector<int>(d.begin(), d.end()), n, upper != 0, attempt, g);
}

}  // namespace

// 0: every check held; > 0: the check that failed; -1: no grid
extern "C" int check_strips(int n, const int* rp, const int* ci, int upper, int attempt) {
  StripGrid g;
  if (!infer(n, rp, ci, upper, attempt, &g)) return -1;
  if (g.nghost > kMaxGhosts || g.dmax > kStripMaxBack) return 9;
  if (const int rc = walk(g, rp, ci, 0 + 1)) return rc;
  return walk(g, rp, ci, kRingSteps - kStripMaxBack);
}

// rows whose level in the grid is not one above the highest of their entries'
extern "C" int check_levels(int n, const int* rp, const int* ci, int upper, int attempt) {
  StripGrid g;
  if (!infer(n, rp, ci, upper, attempt, &g)) return -1;
  int differ = 0;
  for (int i = 0; i < n; ++i) {
    int top = 0;
    for (int e = rp[i]; e < rp[i + 1]; ++e)
      if (ci[e] != i) top = std::max(top, strip_level(g, ci[e]) + 1);
    differ += top != strip_level(g, i);
  }
  return differ;
}

// Estimated times of a solve in strips and row by row (one system repeated
// `systems` times), and the shape: us, us, strips, axis.
extern "C" int strip_costs(int n, const int* rp, const int* ci, int upper, int nlev, int systems,
                           int nrhs, double* out) {
  StripGrid g;
  if (!infer(n, rp, ci, upper, 0, &g)) return -1;
  int max_len = 0;
  for (int i = 0; i < n; ++i) max_len = std::max(max_len, rp[i + 1] - rp[i] - 1);
  const SolveCost c = strip_cost(std::vector<StripGrid>(systems, g), max_len, 8);
  const int64_t rows = static_cast<int64_t>(n) * systems, off = static_cast<int64_t>(rp[n] - n) * systems;
  out[0] = strip_time(c, nrhs);
  out[1] = row_time(rows, off, nlev, max_len, false, nrhs);
  out[2] = c.strips;
  out[3] = g.axis;
  return 0;
}

// Lines of the grid of the given offsets whose run of rows is not what a search
// of every step finds, or -1: no grid.  limit > 0: only so many lines from
// either end, without the search.
extern "C" int check_lines(int n, const int* offsets, int count, int upper, int axis, int limit) {
  StripGrid g;
  if (!strip_infer(std::vector<int>(offsets, offsets + count), n, upper != 0, 0, &g)) return -1;
  g.axis = axis;
  g.stride = axis == 0   ? 1
             : axis == 1 ? g.sy - g.al
                         : g.sz - g.ga * g.sy + g.al * g.ga - g.be;
  if (upper) g.stride = -g.stride;
  const int e1 = g.nx + g.al * (g.ny - 1) + g.be * (g.nz - 1), e2 = g.ny + g.ga * (g.nz - 1);
  const int eu = axis == 0 ? e2 : e1, ev = axis == 2 ? e2 : g.nz, ew = axis == 0 ? e1 : axis == 1 ? e2 : g.nz;
  int wrong = 0;
  for (int v = 0; v < ev; ++v)
    for (int u = 0; u < eu; ++u) {
      if (limit && u >= limit && u < eu - limit) continue;
      int lo, hi;
      strip_line(g, u, v, &lo, &hi);
      if (limit) continue;
      for (int w = 0; w < ew; ++w) {
        const int r = strip_row(g, StripPoint{u, v, w});
        wrong += (r >= 0) != (w >= lo && w < hi);
        if (r >= 0 && w > lo) wrong += r - strip_row(g, StripPoint{u, v, w - 1}) != g.stride;
      }
    }
  return wrong;
}
