// Tiled form of the self-scheduled solve, for triangles whose rows sit on a
// regular grid (Sec. 5.1's model problems and factors with their pattern).
//
// The dependency chain of such a triangle has one link per level, and every
// link of the row-wise schedules is a hop through memory.  Here the rows are
// grouped into tiles of at most 64: boxes of the grid, one lane per row.  A
// wavefront waits once for the values its tile needs from other tiles, then
// solves the tile's own levels through LDS, so a hop is paid per tile of the
// chain and not per row.
//
// Nothing about a pattern is assumed.  The grid's strides are guessed from
// the distinct offsets |i - j| of the entries, and every entry is then
// checked: row i's tile may depend only on tiles that are nowhere ahead of it
// (all three tile coordinates at most its own).  Any map of rows to tiles
// that passes is a valid schedule, whatever the matrix is; a pattern that
// does not pass keeps the row-wise schedules.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <vector>

#include "kernels.hpp"

#if defined(__HIPCC__)
#define SPTRSV_HD __host__ __device__ inline
#else
#define SPTRSV_HD inline
#endif

namespace sptrsv {

// Rows row0 .. row0+n-1 as a grid: row index = x + sy y + sz z, with tiles of
// 2^lx x 2^ly x 2^lz in the skewed coordinates
//   c1 = x + al y + be z,  c2 = y + ga z,  c3 = z
// (the skews keep every dependency from pointing up in any coordinate; 0 for
// the 5- and 7-point stencils).  For an upper triangle x, y, z run backwards.
// The tiles of one (c2, c3) row start at its own first c1, so the boxes
// counted are close to the ones that hold rows.
struct TileGrid {
  int n = 0, row0 = 0;
  int sy = 1, sz = 1;
  int nx = 1, ny = 1, nz = 1;
  int al = 0, be = 0, ga = 0;
  int lx = 6, ly = 0, lz = 0;
  int nbx = 1, nby = 1, nbz = 1;   // boxes along each coordinate
  int box0 = 0;                    // first box of this system
  int upper = 0;
};

struct TilePoint {
  int c1, c2, c3;
};

SPTRSV_HD TilePoint tile_point(const TileGrid& g, int r) {
  int z = r / g.sz;
  const int q = r - z * g.sz;
  int y = q / g.sy;
  int x = q - y * g.sy;
  if (g.upper) {
    x = g.nx - 1 - x;
    y = g.ny - 1 - y;
    z = g.nz - 1 - z;
  }
  return TilePoint{x + g.al * y + g.be * z, y + g.ga * z, z};
}

// row (relative to row0) at a point, or -1
SPTRSV_HD int tile_row(const TileGrid& g, const TilePoint& p) {
  int z = p.c3, y = p.c2 - g.ga * z, x = p.c1 - g.al * y - g.be * z;
  if (x < 0 || x >= g.nx || y < 0 || y >= g.ny || z < 0 || z >= g.nz) return -1;
  if (g.upper) {
    x = g.nx - 1 - x;
    y = g.ny - 1 - y;
    z = g.nz - 1 - z;
  }
  const int64_t r = x + static_cast<int64_t>(g.sy) * y + static_cast<int64_t>(g.sz) * z;
  return r < g.n ? static_cast<int>(r) : -1;
}

SPTRSV_HD int tile_first_y(const TileGrid& g, int t3) { return (g.ga * (t3 << g.lz)) >> g.ly; }

SPTRSV_HD int tile_first_x(const TileGrid& g, int t2, int t3) {
  return (g.al * (t2 << g.ly) + (g.be - g.al * g.ga) * (t3 << g.lz)) >> g.lx;
}

// box of a point, and its lane inside the box
SPTRSV_HD int tile_box(const TileGrid& g, const TilePoint& p) {
  const int t1 = p.c1 >> g.lx, t2 = p.c2 >> g.ly, t3 = p.c3 >> g.lz;
  return (t3 * g.nby + (t2 - tile_first_y(g, t3))) * g.nbx + (t1 - tile_first_x(g, t2, t3));
}

SPTRSV_HD int tile_lane(const TileGrid& g, const TilePoint& p) {
  const int u = p.c1 & ((1 << g.lx) - 1), v = p.c2 & ((1 << g.ly) - 1),
            w = p.c3 & ((1 << g.lz) - 1);
  return u | (v << g.lx) | (w << (g.lx + g.ly));
}

// tile coordinates of a box (the inverse of tile_box)
SPTRSV_HD TilePoint tile_of_box(const TileGrid& g, int box) {
  const int t3 = box / (g.nbx * g.nby);
  const int q = box - t3 * g.nbx * g.nby;
  const int b2 = q / g.nbx;
  const int t2 = b2 + tile_first_y(g, t3);
  return TilePoint{q - b2 * g.nbx + tile_first_x(g, t2, t3), t2, t3};
}

// the point of a lane of a box
SPTRSV_HD TilePoint tile_lane_point(const TileGrid& g, const TilePoint& t, int lane) {
  const int u = lane & ((1 << g.lx) - 1), v = (lane >> g.lx) & ((1 << g.ly) - 1),
            w = lane >> (g.lx + g.ly);
  return TilePoint{(t.c1 << g.lx) | u, (t.c2 << g.ly) | v, (t.c3 << g.lz) | w};
}

constexpr int kTileMaxOffsets = 13;   // distinct offsets of a pattern (27-point stencil)
constexpr int kTileTable = 32;        // slots of the device's offset table per system
constexpr int kTileMaxEntries = 16;   // entry slots of a row
constexpr int kTileMaxExt = 191;      // values a tile may need from others (8-bit slots)

// Guesses the grid of one system from its distinct offsets (ascending) and
// picks the tile shape.  `attempt` 0, 1 choose between the readings of an
// offset cluster of even width.  *ext: values a full tile needs from others.
// false: no grid.
bool tile_infer(const std::vector<int>& offsets, int n, bool upper, int attempt, TileGrid* g,
                int* ext);

// Tiled copy of one triangle.  Positions are tile * 64 + lane; lanes without
// a row exist in tiles at the grid's edges.
struct DevTiles {
  int ntiles = 0;
  int order = 1;            // steps of the tile order (sums of tile coordinates)
  int entries = 0;          // entry slots per row (E)
  int ext = 0;              // words of external positions per lane (X)
  int acc = 1;              // partial sums per row: 1, or 4 (see k_tile)
  int64_t npos = 0;         // ntiles * 64
  int* row = nullptr;       // [npos] caller's row | log2(partial sums) << 30; -1: no row
  int* depth = nullptr;     // [ntiles] levels inside the tile
  unsigned* slot = nullptr; // [ntiles][(E+3)/4][64] LDS slots of the entries, four per word
  int* epos = nullptr;      // [ntiles][X][64] positions of the external values, -1: none
  int* src = nullptr;       // [ntiles][E][64] value of the entry in the plan, -1: no entry
  int* dsrc = nullptr;      // [npos] position in the plan (1/diagonal)
  void* val = nullptr;      // [ntiles][E][64] T
  void* dinv = nullptr;     // [npos] T
  void* mem = nullptr;      // the one allocation behind all of these
};

// Distinct offsets of every system: table[s * kTileTable ..], 0 = empty;
// full[s] != 0: more than kTileMaxOffsets.  Rows of the systems are
// sys_row0[0 .. nsys].  row_ptr / col: CSR of the whole triangle.
hipError_t launch_tile_offsets(int n, const int* row_ptr, const int* col, int nsys,
                               const int* sys_row0, int* table, int* full, hipStream_t s);

// Builds the tiled copy of plan p (values excluded) for the given grids.
// Returns kOk, kErrNotSupported (some entry does not fit the grids, or a tile
// needs more than 8-bit slots), kErrOom or kErrHip; nothing is kept on
// failure.  lanes_lg: log2 of the lanes the row-wise schedules give the row at
// each position (null: one lane everywhere); max_len: longest row.
// Blocking.
int build_tiles(const DevPlan& p, const std::vector<TileGrid>& grids, int ext, int max_len,
                const unsigned char* lanes_lg, int vb, hipStream_t s, DevTiles& out);
void free_tiles(DevTiles& t);

// lanes_lg[k] for a chunk table
hipError_t launch_tile_lanes(const DevChunks& c, unsigned char* lanes_lg, hipStream_t s);

// values of the tiled copy from the plan's
template <typename T> hipError_t launch_tile_gather(const DevPlan& p, const DevTiles& t,
                                                    hipStream_t s);

struct TileSolveArgs {
  const DevTiles* tiles;
  DevScratch scratch;
  const void* b;
  void* x;
  void* xp;          // [npos] published values, filled with the sentinel
  int spin_limit = 1 << 22;
  int res_limit = 1 << 20;
  int coop = 0;
  int grid = 1;      // one-wavefront workgroups, all resident
};
template <typename T> hipError_t launch_tile_solve(const TileSolveArgs& a, hipStream_t s);
template <typename T> int tile_blocks_per_cu(const DevTiles& t);

}  // namespace sptrsv
