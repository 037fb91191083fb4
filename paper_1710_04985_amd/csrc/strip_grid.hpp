// Geometry of the strip form (strips.hpp): grids, strips and their lines.
// Plain C++, no HIP calls.
#pragma once

#include <cstdint>
#include <vector>

#if defined(__HIPCC__)
#define SPTRSV_HD __host__ __device__ inline
#else
#define SPTRSV_HD inline
#endif

namespace sptrsv {

constexpr int kRingSteps = 16;         // steps the LDS ring holds
constexpr int kDumpSlot = 16;          // values between the strips' lines for what nobody reads
constexpr int kStripMaxBack = 7;       // steps an entry may reach back
constexpr int kRingCols = 128;         // its columns: lanes, ghosts, and the zero column
constexpr int kZeroCol = 127;
constexpr int kMaxGhosts = 63;
constexpr int kStripMaxSteps = 1 << 17;  // steps of a strip
constexpr int kStripMaxOffsets = 13;   // distinct offsets of a pattern (27-point stencil)
constexpr int kStripTable = 32;        // slots of the device's offset table per system
constexpr int kStripMaxEntries = 16;   // entry slots of a row

// Rows row0 .. row0+n-1 as a grid: row index = x + sy y + sz z, in the skewed
// coordinates
//   c1 = x + al y + be z,  c2 = y + ga z,  c3 = z
// (the skews keep every dependency from pointing up in any coordinate; 0 for
// the 5- and 7-point stencils).  For an upper triangle x, y, z run backwards.
// A strip walks along coordinate `axis` (0: c1, 1: c2, 2: c3); its lanes are a
// 2^lu x 2^lv box of the other two, in order.
struct StripGrid {
  int n = 0, row0 = 0;
  int sy = 1, sz = 1;
  int nx = 1, ny = 1, nz = 1;
  int al = 0, be = 0, ga = 0;
  int wx = 0, wy = 0, wz = 0;   // the level of (x, y, z) in a grid without gaps
  int upper = 0;
  int axis = 0, lu = 6, lv = 0;
  int nbu = 1, nbv = 1;      // strips along the two lane coordinates
  int box0 = 0;              // first box of this system
  int stride = 1;            // row index step along the lines
  int dmax = 1;              // steps back of the farthest dependency
  int gu = 0, gv = 0;        // lines back of the farthest dependency, per lane coordinate
  double chain = 0, work = 0;   // steps of the longest chain of strips (a hop counts
                             // as ten), and of all strips: estimates
  int npub = 0;              // lanes that other strips read
  int nghost = 0;            // lines of other strips that a strip reads
  // ghost of a line outside the strip: ghost[(u + gu) + (v + gv) * (2^lu + gu)],
  // 255 = none
  unsigned char ghost[256];
  unsigned char gcol[64];    // its inverse: the index above of ghost g
  signed char pub[64];       // place of a lane among the published ones, -1 = not published
};

// wx x + wy y + wz z of a row (relative to row0): its level, if every row of the grid
// has all the entries that fit
SPTRSV_HD int strip_level(const StripGrid& g, int r) {
  const int z = r / g.sz;
  const int q = r - z * g.sz;
  const int y = q / g.sy;
  const int x = q - y * g.sy;
  return g.upper ? g.wx * (g.nx - 1 - x) + g.wy * (g.ny - 1 - y) + g.wz * (g.nz - 1 - z)
                 : g.wx * x + g.wy * y + g.wz * z;
}

struct StripPoint {
  int u, v, w;   // lane coordinates and the coordinate along the lines
};

SPTRSV_HD StripPoint strip_point(const StripGrid& g, int r) {
  int z = r / g.sz;
  const int q = r - z * g.sz;
  int y = q / g.sy;
  int x = q - y * g.sy;
  if (g.upper) {
    x = g.nx - 1 - x;
    y = g.ny - 1 - y;
    z = g.nz - 1 - z;
  }
  const int c1 = x + g.al * y + g.be * z, c2 = y + g.ga * z;
  return g.axis == 0 ? StripPoint{c2, z, c1}
                     : g.axis == 1 ? StripPoint{c1, z, c2} : StripPoint{c1, c2, z};
}

// row index (relative to row0) of a point, which may lie outside the grid: linear
// in its coordinates; *inside: whether it lies in the grid, its last plane and
// line taken to be whole
SPTRSV_HD int64_t strip_index(const StripGrid& g, const StripPoint& p, bool* inside) {
  const int64_t c1 = g.axis == 0 ? p.w : p.u;
  const int64_t c2 = g.axis == 0 ? p.u : g.axis == 1 ? p.w : p.v;
  int64_t z = g.axis == 2 ? p.w : p.v;
  int64_t y = c2 - g.ga * z, x = c1 - g.al * y - g.be * z;
  *inside = x >= 0 && x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz;
  if (g.upper) {
    x = g.nx - 1 - x;
    y = g.ny - 1 - y;
    z = g.nz - 1 - z;
  }
  return x + g.sy * y + g.sz * z;
}

// row (relative to row0) at a point, or -1
SPTRSV_HD int strip_row(const StripGrid& g, const StripPoint& p) {
  bool inside;
  const int64_t r = strip_index(g, p, &inside);
  return inside && r < g.n ? static_cast<int>(r) : -1;
}

// [lo, hi) := the w in it with 0 <= k w + m < N
SPTRSV_HD void strip_clip(int64_t k, int64_t m, int64_t N, int64_t* lo, int64_t* hi) {
  if (k == 0) {
    if (m < 0 || m >= N) *hi = *lo;
    return;
  }
  // for k < 0 mirror the condition: 0 <= -k w + (N - 1 - m) < N
  if (k < 0) {
    k = -k;
    m = N - 1 - m;
  }
  const int64_t a = -m, b = N - m;                     // a <= k w < b
  const int64_t l = a >= 0 ? (a + k - 1) / k : -((-a) / k);
  const int64_t h = b > 0 ? (b + k - 1) / k : -((-b) / k);
  if (l > *lo) *lo = l;
  if (h < *hi) *hi = h;
  if (*hi < *lo) *hi = *lo;
}

// The w with a row on line (u, v): one run [lo, hi), since all conditions are
// linear in w.
SPTRSV_HD void strip_line(const StripGrid& g, int u, int v, int* lo_out, int* hi_out) {
  int64_t lo = 0, hi = 1ll << 30;
  const int64_t al = g.al, be = g.be, ga = g.ga;
  if (u < 0 || v < 0) {
    hi = 0;
  } else if (g.axis == 0) {            // u = c2, v = z
    const int64_t z = v, y = u - ga * z;
    strip_clip(0, z, g.nz, &lo, &hi);
    strip_clip(0, y, g.ny, &lo, &hi);
    strip_clip(1, -al * y - be * z, g.nx, &lo, &hi);
  } else if (g.axis == 1) {            // u = c1, v = z, w = c2: y = w - ga z
    const int64_t z = v;
    strip_clip(0, z, g.nz, &lo, &hi);
    strip_clip(1, -ga * z, g.ny, &lo, &hi);
    strip_clip(-al, u + al * ga * z - be * z, g.nx, &lo, &hi);
  } else {                             // u = c1, v = c2, w = z
    strip_clip(1, 0, g.nz, &lo, &hi);
    strip_clip(-ga, v, g.ny, &lo, &hi);
    strip_clip(al * ga - be, u - al * static_cast<int64_t>(v), g.nx, &lo, &hi);
  }
  // the last line or plane may be cut off by n: the row at w is linear in it
  if (lo < hi) {
    bool inside;
    const int64_t first = strip_index(g, StripPoint{u, v, static_cast<int>(lo)}, &inside);
    strip_clip(g.stride, first - lo * g.stride, g.n, &lo, &hi);
  }
  *lo_out = static_cast<int>(lo);
  *hi_out = static_cast<int>(hi);
}

// Guesses the grid of one system from its distinct offsets (ascending) and
// picks the strips' shape.  `attempt` 0, 1 choose between the readings of an
// offset cluster of even width.  false: no grid.
bool strip_infer(const std::vector<int>& offsets, int n, bool upper, int attempt, StripGrid* g);

// What decides between the strip form and the row-wise schedules.
struct SolveCost {
  double chain = 0;          // steps of the longest chain, over all systems
  double strips = 0, work = 0;   // strips, and their steps, of all systems
  int words = 0;             // 32-bit words of a lane's record
};
SolveCost strip_cost(const std::vector<StripGrid>& grids, int max_len, int vb);

// Estimated time of a solve in strips, and row by row (block: by the block
// schedule), in us.
double strip_time(const SolveCost& c, int nrhs);
double row_time(int64_t n, int64_t noff, int nlev, int max_len, bool block, int nrhs);

}  // namespace sptrsv
