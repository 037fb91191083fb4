// Strip form of the self-scheduled solve, for triangles whose rows sit on a
// regular grid (Sec. 5.1's model problems and factors with their pattern).
//
// The dependency chain of such a triangle has one link per level, and every
// link of the row-wise schedules is a hop through memory.  Here the grid is
// cut into strips: up to 64 neighbouring grid lines, one line per lane of a
// wavefront, walked along the lines with one step's skew between neighbouring
// lanes.  A row's dependencies are then rows that the same wavefront solved a
// few steps earlier, kept in an LDS ring, or rows of neighbouring strips,
// whose values stream in through memory as they are published.  A hop is paid
// once per strip of the chain, not once per level.
//
// Nothing about a pattern is assumed.  The grid's strides are guessed from
// the distinct offsets |i - j| of the entries, and every entry is then
// checked: it must lead to an earlier step of its own strip, or to a strip
// that is earlier in the order (no coordinate ahead of its own), at a place
// the ring holds.  Any pattern that does not pass keeps the row-wise
// schedules, and so does one whose levels are few and wide for the length of
// its lines (strip_time against row_time, strip_grid.hpp).
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <vector>

#include "kernels.hpp"
#include "strip_grid.hpp"

namespace sptrsv {

// Strip-ordered copy of one triangle.  Strip p takes `steps` records of 64
// lanes; a lane's record holds the row's entry values, 1/diagonal and the
// ring addresses of its entries (16 bits each), as words.  Word w < 4 * (words
// / 4) of lane l in record r sits at quad[(r * (words / 4) + w / 4) * 64 + l];
// the remaining words at tail[(r * 64 + l) * (words % 4)].
struct StripInfo {
  int steps;
  int stride;      // row index step
  int npub;        // published lanes per step
  int ghost_lg;    // log2 of the ghost lines, rounded up; -1: none
  int64_t rec0;    // first record
  int64_t pub0;    // first published value
};

struct StripLane {
  int row0;        // row at step s: row0 + s * stride, for lo <= s < lo + len
  int lo, len;
  int rlo, rhi;  // first and last such step of any of the eight lanes 8 (l / 8) ..
  int pub;         // place among the strip's published lanes, or -1
  int glo, glen;   // the lane's ghost line has values for glo <= s < glo + glen
  int64_t gpos;    // published value of the ghost at step s: gpos + s * npub
};

struct DevStrips {
  int nstrips = 0;
  int entries = 0;          // entry slots per row (E)
  int acc = 1;              // partial sums per row: 1, or 4 (see k_strip)
  int words = 0;            // words of a record
  int64_t nrec = 0;         // records
  int64_t npub = 0;         // published values
  StripInfo* info = nullptr;    // [nstrips]
  StripLane* lane = nullptr;    // [nstrips][64]
  void* quad = nullptr;
  unsigned* tail = nullptr;
  int* src = nullptr;       // [nrec][E][64] value of the entry in the plan, -1: no entry
  int* dsrc = nullptr;      // [nrec][64] position in the plan, -1: no row
  void* mem = nullptr;      // the one allocation behind all of these
};

// Distinct offsets of every system: table[s * kStripTable ..], 0 = empty;
// full[s] != 0: more than the table holds.  Rows of the systems are
// sys_row0[0 .. nsys].  row_ptr / col: CSR of the whole triangle, which need not have
// been checked yet (what is read stays in bounds).
hipError_t launch_strip_offsets(int n, int64_t nnz, const int* row_ptr, const int* col,
                                int nsys, const int* sys_row0, int* table, int* full,
                                hipStream_t s);

// Builds the strip-ordered copy of plan p (values excluded) for the given
// grids.  Returns kOk, kErrNotSupported (some entry does not fit the grids),
// kErrOom or kErrHip; nothing is kept on failure.  lanes_lg: log2 of the lanes
// the row-wise schedules give the row at each position (null: one lane
// everywhere); max_len: longest row.  Blocking.
int build_strips(const DevPlan& p, const std::vector<StripGrid>& grids, int max_len,
                 const unsigned char* lanes_lg, int vb, hipStream_t s, DevStrips& out);
void free_strips(DevStrips& t);

// lanes_lg[k] for a chunk table
hipError_t launch_strip_lanes(const DevChunks& c, unsigned char* lanes_lg, hipStream_t s);

// values of the strip-ordered copy from the plan's
template <typename T> hipError_t launch_strip_gather(const DevPlan& p, const DevStrips& t,
                                                     hipStream_t s);

// values of the solution buffer a solve uses; the first npub * nrhs of them are
// filled with the sentinel before it
inline int64_t strip_values(const DevStrips& t, int nrhs) {
  return (t.npub + static_cast<int64_t>(kDumpSlot) * t.nstrips) * nrhs;
}

// The kernel's partial sums of a row: several right-hand sides are computed as
// the one-lane solve computes each.
inline int strip_sums(const DevStrips& t, int nrhs) { return nrhs > 1 ? 1 : t.acc; }

// Stages of records that the kernel holds (it loads them depth - 1 steps
// ahead), for values of vb bytes.  Long records, loaded 7 steps ahead instead
// of 3: faster where they come from memory, but in FP64 the extra stages sit in
// accumulation registers, so a step has more to do.  27-point, FP64, us per
// solve at 7 / 3 steps, two triangles in turn (which push each other out of the
// 256 MB cache from 128 MB each on): 68^3 (87 MB of records) 164 / 153, 80^3 (123)
// 194 / 185, 82^3 (135) 208 / 209, 85^3 (152) 223 / 229, 95^3 (197) 267 / 282;
// one triangle alone 95^3 234 / 224.  Several columns reach memory sooner: four, in
// turn, 68^3 156 / 156, 76^3 (107 MB) 177 / 178, 80^3 191 / 196.  FP32, both
// triangles: 20^3 90 / 91, 60x50x40 183 / 190, 128^3 576 / 688.
inline int strip_depth(const DevStrips& t, int vb, int nrhs) {
  if (t.entries <= 4) return 16;
  return vb == 4 || t.nrec * t.words * 256 > (nrhs > 1 ? 100 << 20 : 128 << 20) ? 8 : 4;
}

struct StripSolveArgs {
  const DevStrips* strips;
  DevScratch scratch;
  const void* b;
  void* x;
  void* xp;          // [strip_values]
  int nrhs = 1;
  int64_t ld = 0;    // elements between the columns of b and x
  int spin_limit = 1 << 22;
  int grid = 1;      // four-wavefront workgroups
};
template <typename T> hipError_t launch_strip_solve(const StripSolveArgs& a, hipStream_t s);
template <typename T> int strip_blocks_per_cu(const DevStrips& t, int nrhs);

}  // namespace sptrsv
