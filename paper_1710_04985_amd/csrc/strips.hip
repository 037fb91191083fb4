// Strip-wise self-scheduled solve: construction of the strip-ordered copy, and
// the solve kernel (see strips.hpp for the idea).
#include "strips.hpp"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "analysis.hpp"
#include "device_common.hpp"
#include "devmem.hpp"

namespace sptrsv {
namespace {

constexpr int kRecordThreads = 256;

// ------------------------------------------------------------ construction

// System of a row: the last s with row0[s] <= i.
__device__ __forceinline__ int system_of(const int* __restrict__ row0, int nsys, int i) {
  int lo = 0, hi = nsys - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (row0[mid] <= i) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Adds d > 0 to an open-addressed table of kStripTable slots; false: no room.
__device__ __forceinline__ bool table_add(int* table, int d, bool agent) {
  unsigned h = (static_cast<unsigned>(d) * 2654435761u) >> 27;
  for (int probe = 0; probe < kStripTable; ++probe, h = (h + 1) & (kStripTable - 1)) {
    int v = agent ? __hip_atomic_load(table + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                  : __hip_atomic_load(table + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (v == d) return true;
    if (v == 0) {
      v = atomicCAS(table + h, 0, d);
      if (v == 0 || v == d) return true;
    }
  }
  return false;
}

// Each workgroup collects the offsets of a contiguous run of rows in LDS,
// system by system, and then adds the few distinct ones to the system's
// table, so that global atomics do not grow with the entries.  Runs are short
// enough for 512 workgroups (13,824 rows of 13 entries: 70 us in runs of 4096,
// 9 in runs of 256), and for twice as many where systems, which follow one
// another in a run, about 2 us each, may be small (4000 systems of 4 rows, whole
// set-up: 4.7 ms in runs of 4096, 0.5 before there were strips).
inline int offset_rows(int n, int nsys) {
  return nsys == 1 ? std::min(std::max(n / 512, 256), 4096) : std::min(std::max(n / 1024, 64), 4096);
}

__global__ void __launch_bounds__(256)
k_strip_offsets(int n, int64_t nnz, const int* __restrict__ rp, const int* __restrict__ col, int nsys,
               const int* __restrict__ row0, int rows, int* table, int* full) {
  __shared__ int tab[kStripTable];
  __shared__ int over;
  const int r0 = blockIdx.x * rows, r1 = min(n, r0 + rows);
  int s = system_of(row0, nsys, r0);
  for (int a = r0; a < r1; ++s) {
    const int b = min(r1, row0[s + 1]);
    if (threadIdx.x < kStripTable) tab[threadIdx.x] = 0;
    if (threadIdx.x == 0) over = 0;
    __syncthreads();
    for (int i = a + threadIdx.x; i < b && !over; i += 256) {
      int e = rp[i], e1 = rp[i + 1];
      if (e < 0 || e1 > nnz) e1 = e;        // not a valid pattern: the checks refuse it
      for (; e < e1; ++e) {
        const int d = abs(col[e] - i);
        if (d != 0 && !table_add(tab, d, false)) {
          over = 1;
          break;
        }
      }
    }
    __syncthreads();
    if (threadIdx.x < kStripTable) {
      const int d = tab[threadIdx.x];
      if (over || (d != 0 && !table_add(table + static_cast<int64_t>(s) * kStripTable, d, true)))
        __hip_atomic_store(full + s, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    a = b;
  }
}

__global__ void __launch_bounds__(256)
k_strip_lanes(int nchunks, const int* __restrict__ start, const int* __restrict__ meta,
             unsigned char* __restrict__ lanes_lg) {
  const int c = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, lane = threadIdx.x & 63;
  if (c >= nchunks) return;
  const int cnt = meta[c] & 0xffff, lg = meta[c] >> 16;
  for (int r = lane; r < cnt; r += 64) lanes_lg[start[c] + r] = static_cast<unsigned char>(lg);
}

// slot of entry e of a row with 2^lg partial sums (see k_strip)
__device__ __forceinline__ int entry_slot(int e, int lg, int acc) {
  return acc == 1 ? e : 4 * (e >> lg) + (e & ((1 << lg) - 1));
}

// Place of a record's word: quads of four words are loaded 16 bytes per lane,
// the rest as one short load.
__device__ __forceinline__ unsigned* word_at(const DevStrips& d, int64_t rec, int lane, int w) {
  const int nq = d.words / 4, nt = d.words % 4;
  return w < 4 * nq
             ? static_cast<unsigned*>(d.quad) + ((rec * nq + (w >> 2)) * 64 + lane) * 4 + (w & 3)
             : d.tail + (rec * 64 + lane) * nt + (w - 4 * nq);
}

// counters of the construction
struct StripCount {
  int bad;                  // an entry does not fit the grids
  int slots;                // entry slots a row needs
  unsigned long long rows;  // rows on lines
};

// One wavefront per box: the first step that holds rows, less the steps the
// farthest dependency reaches back (so every step read from the ring is one
// of the strip's own), and the number of steps (0: no rows).
__global__ void __launch_bounds__(64)
k_strip_boxes(const StripGrid* __restrict__ grids, int nsys, const int* __restrict__ sys_box0,
              int2* __restrict__ out, StripCount* cnt) {
  const int box = blockIdx.x, lane = threadIdx.x;
  const StripGrid& g = grids[nsys > 1 ? system_of(sys_box0, nsys, box) : 0];
  const int q = box - g.box0, bv = q / g.nbu, bu = q - bv * g.nbu;
  const int u = (bu << g.lu) + (lane & ((1 << g.lu) - 1)), v = (bv << g.lv) + (lane >> g.lu);
  int lo, hi;
  strip_line(g, u, v, &lo, &hi);
  int first = hi > lo ? lo + u + v : INT32_MAX, end = hi > lo ? hi + u + v : INT32_MIN;
  int rows = hi - lo;
  for (int o = 32; o > 0; o >>= 1) {
    first = min(first, __shfl_xor(first, o, 64));
    end = max(end, __shfl_xor(end, o, 64));
    rows += __shfl_xor(rows, o, 64);
  }
  if (lane == 0) {
    out[box] = rows > 0 ? make_int2(first - g.dmax, end - (first - g.dmax)) : make_int2(0, 0);
    if (rows > 0) atomicAdd(&cnt->rows, static_cast<unsigned long long>(rows));
  }
}

// entry slots the row that needs most needs, with four partial sums
__global__ void __launch_bounds__(256)
k_strip_slots(int n, const int* __restrict__ off_ptr, const unsigned char* __restrict__ lanes_lg,
              StripCount* cnt) {
  int slots = 0;
  const int stride = gridDim.x * blockDim.x;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += stride) {
    const int len = off_ptr[k + 1] - off_ptr[k], lg = lanes_lg[k];
    if (len > 0) slots = max(slots, lg > 2 ? kStripMaxEntries + 1 : entry_slot(len - 1, lg, 4) + 1);
  }
  for (int o = 32; o > 0; o >>= 1) slots = max(slots, __shfl_xor(slots, o, 64));
  if ((threadIdx.x & 63) == 0 && slots) atomicMax(&cnt->slots, slots);
}

// what a strip is cut from
struct StripBox {
  int sys, bu, bv, first;
};

// One wavefront per strip: its lanes' rows and ghost lines.
__global__ void __launch_bounds__(64)
k_strip_lanes_of(const StripGrid* __restrict__ grids, const StripBox* __restrict__ boxes,
                 const int* __restrict__ box_strip, DevStrips d, StripCount* cnt) {
  const int p = blockIdx.x, lane = threadIdx.x;
  const StripBox bx = boxes[p];
  const StripGrid& g = grids[bx.sys];
  const StripInfo inf = d.info[p];
  const int TU = 1 << g.lu;
  const int u = (bx.bu << g.lu) + (lane & (TU - 1)), v = (bx.bv << g.lv) + (lane >> g.lu);
  StripLane l;
  int lo, hi;
  strip_line(g, u, v, &lo, &hi);
  l.lo = hi > lo ? lo + u + v - bx.first : 0;
  l.len = hi - lo;
  // a lane without rows reads the system's first row over and over
  l.row0 = g.row0 + (hi > lo ? strip_row(g, StripPoint{u, v, lo}) - l.lo * g.stride : 0);
  // a cache line of a record holds eight lanes: they stay together
  l.rlo = hi > lo ? l.lo : INT32_MAX;
  l.rhi = hi > lo ? l.lo + l.len - 1 : 0;
  for (int o = 1; o < 8; o <<= 1) {
    l.rlo = min(l.rlo, __shfl_xor(l.rlo, o, 64));
    l.rhi = max(l.rhi, __shfl_xor(l.rhi, o, 64));
  }
  l.rlo = min(l.rlo, l.rhi);
  l.pub = g.pub[lane];
  l.glo = l.glen = 0;
  l.gpos = 0;
  bool bad = false;
  if (lane < g.nghost) {
    const int q = g.gcol[lane], W = TU + g.gu;
    const int gu = (bx.bu << g.lu) + q % W - g.gu, gv = (bx.bv << g.lv) + q / W - g.gv;
    if (gu >= 0 && gv >= 0) {
      const int p2 = box_strip[g.box0 + (gv >> g.lv) * g.nbu + (gu >> g.lu)];
      strip_line(g, gu, gv, &lo, &hi);
      if (p2 >= 0 && hi > lo) {
        const int from = g.pub[(gu & (TU - 1)) | ((gv & ((1 << g.lv) - 1)) << g.lu)];
        bad = from < 0 || p2 >= p;
        l.glo = lo + gu + gv - bx.first;
        l.glen = hi - lo;
        l.gpos = d.info[p2].pub0 +
                 static_cast<int64_t>(bx.first - boxes[p2].first) * inf.npub + max(from, 0);
      }
    }
  }
  d.lane[static_cast<int64_t>(p) * 64 + lane] = l;
  if (__any(bad) && lane == 0) atomicOr(&cnt->bad, 1);
}

// Ring addresses and value sources of the rows of one record (step s of strip
// p), by one wavefront.
__device__ __forceinline__ void
strip_record(const int* __restrict__ off_ptr, const int* __restrict__ off_col,
             const int* __restrict__ row_pos, const unsigned char* __restrict__ lanes_lg,
             const StripGrid* __restrict__ grids, const StripBox* __restrict__ boxes, int vb,
             const DevStrips& d, StripCount* cnt, int p, int s, const StripInfo& inf) {
  const int lane = threadIdx.x & 63;
  const StripBox bx = boxes[p];
  const StripGrid& g = grids[bx.sys];
  const StripLane l = d.lane[static_cast<int64_t>(p) * 64 + lane];
  const int64_t rec = inf.rec0 + s;
  const int E = d.entries, TU = 1 << g.lu, TV = 1 << g.lv;
  const int u0 = bx.bu << g.lu, v0 = bx.bv << g.lv;
  const bool act = static_cast<unsigned>(s - l.lo) < static_cast<unsigned>(l.len);
  const int r = act ? l.row0 + s * g.stride - g.row0 : -1;
  bool bad = false;
  int k = -1;
  if (act) {
    const int u = u0 + (lane & (TU - 1)), v = v0 + (lane >> g.lu);
    bad = r < 0 || r >= g.n;
    if (!bad) {
      const StripPoint q = strip_point(g, r);
      bad = q.u != u || q.v != v || q.w != s + bx.first - u - v;
    }
    if (!bad) k = row_pos[g.row0 + r];
  }
  for (int q = 0; q < E; ++q) d.src[(rec * E + q) * 64 + lane] = -1;
  d.dsrc[rec * 64 + lane] = k;
  if (k >= 0) {
    const int e0 = off_ptr[k], len = off_ptr[k + 1] - e0;
    const int lg = lanes_lg ? lanes_lg[k] : 0;
    const int cw = (E + 1) * (vb / 4);
    constexpr int kHalves = kStripMaxEntries + 2;
    unsigned short code[kHalves];
#pragma unroll
    for (int q = 0; q < kHalves; ++q) code[q] = static_cast<unsigned short>(kZeroCol * vb);
    for (int e = 0; e < len; ++e) {
      const int j = off_col[e0 + e] - g.row0;
      const int q = entry_slot(e, lg, d.acc);
      if (j < 0 || j >= g.n || q >= E) {
        bad = true;
        break;
      }
      const StripPoint t = strip_point(g, j);
      const int back = s - (t.u + t.v + t.w - bx.first), du = t.u - u0, dv = t.v - v0;
      int col = -1;
      if (du >= 0 && dv >= 0 && du < TU && dv < TV) {
        col = du | (dv << g.lu);
      } else if (du >= -g.gu && dv >= -g.gv && du < TU && dv < TV) {
        const int gh = g.ghost[(du + g.gu) + (dv + g.gv) * (TU + g.gu)];
        if (gh < kMaxGhosts) col = 64 + gh;
      }
      if (col < 0 || back < 1 || back > g.dmax) {
        bad = true;
        break;
      }
#pragma unroll
      for (int h = 0; h < kHalves; ++h)
        if (h == q) code[h] = static_cast<unsigned short>(((((s - back) & (kRingSteps - 1)) << 7) | col) * vb);
      d.src[(rec * E + q) * 64 + lane] = e0 + e;
    }
    // with four partial sums the spare half word holds the row's own count
#pragma unroll
    for (int h = 0; h < kHalves; ++h)
      if (d.acc == 4 && h == E) code[h] = static_cast<unsigned short>(lg);
#pragma unroll
    for (int h = 0; h < kHalves; h += 2)
      if (h < E) *word_at(d, rec, lane, cw + h / 2) = code[h] | (static_cast<unsigned>(code[h + 1]) << 16);
  }
  if (__any(bad) && lane == 0) atomicOr(&cnt->bad, 1);
}

// Workgroups per strip: four steps each, and all of the longest strip's at once
// unless the strips' lengths differ so much that most workgroups would find
// nothing to do (a batch of many small systems and one long chain); the long
// ones' then take several turns.  (One wavefront per four records in a row,
// its strip searched for: 128^3 set-up 1.36 ms against 1.32.)
constexpr int kRecordWaves = kRecordThreads / 64;

inline unsigned record_blocks(int64_t nrec, int nstrips, int max_steps) {
  const int64_t all = (max_steps + kRecordWaves - 1) / kRecordWaves;
  const int64_t fair = std::max<int64_t>(4 * nrec / nstrips / kRecordWaves + 1, 65536 / nstrips + 1);
  return static_cast<unsigned>(std::min(all, fair));
}

// (a loop around the one turn that most triangles take cost it a sixth)
template <bool kTurns>
__global__ void __launch_bounds__(kRecordThreads)
k_strip_records(const int* __restrict__ off_ptr, const int* __restrict__ off_col,
                const int* __restrict__ row_pos, const unsigned char* __restrict__ lanes_lg,
                const StripGrid* __restrict__ grids, const StripBox* __restrict__ boxes, int vb,
                DevStrips d, StripCount* cnt) {
  const int p = blockIdx.x;
  int s = blockIdx.y * kRecordWaves + (threadIdx.x >> 6);
  const StripInfo inf = d.info[p];
  if (s >= inf.steps) return;
  do {
    strip_record(off_ptr, off_col, row_pos, lanes_lg, grids, boxes, vb, d, cnt, p, s, inf);
    if constexpr (kTurns) s += gridDim.y * kRecordWaves;
  } while (kTurns && s < inf.steps);
}

// values of the strip-ordered copy: entries a row lacks are -0, whose product
// with the zero column (+0) is -0 and changes no sum
template <typename T>
__global__ void __launch_bounds__(256)
k_strip_gather(DevStrips d, const T* __restrict__ off_val, const T* __restrict__ dinv) {
  constexpr int VW = sizeof(T) / 4;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= d.nrec * 64) return;
  const int64_t rec = t >> 6;
  const int lane = static_cast<int>(t & 63);
  const int k = d.dsrc[t];
  if (k < 0) return;
  for (int q = 0; q <= d.entries; ++q) {
    T v;
    if (q < d.entries) {
      const int s = d.src[(rec * d.entries + q) * 64 + lane];
      v = s >= 0 ? off_val[s] : -T(0);
    } else {
      v = dinv[k];
    }
    unsigned w[VW];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int h = 0; h < VW; ++h) *word_at(d, rec, lane, q * VW + h) = w[h];
  }
}

// -------------------------------------------------------------------- solve

template <typename T> struct SArgs {
  int nstrips;
  int nrhs;
  int64_t ld;        // elements between the columns of b and x
  int64_t npub;
  const StripInfo* info;
  const StripLane* lane;
  const char* quad;
  const char* tail;
  const T* b;
  T* x;
  T* xp;
  int* status;
  int* ticket;       // 0 at the start (the sentinel fill's counter)
  int spin_limit;
};

template <int N> struct Words {
  unsigned w[N];
};

__device__ __forceinline__ int64_t uniform64(int64_t v) {
  return static_cast<int64_t>(static_cast<unsigned>(wave_uniform(static_cast<int>(v)))) |
         static_cast<int64_t>(wave_uniform(static_cast<int>(v >> 32))) << 32;
}

// What the wavefronts of a strip tell each other (in LDS): steps whose ghost
// values, and whose b, are in place; steps solved; steps taken over for
// storing.  The LDS performs a wavefront's accesses in issue order, so a
// counter written after the data is seen after the data; the fences order the
// compiler only.
struct StripCounters {
  int avail, bready, done, stored, strip;
};

__device__ __forceinline__ int read_counter(const int* c) {
  const int v = wave_uniform(
      __hip_atomic_load(const_cast<int*>(c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  return v;
}

__device__ __forceinline__ void write_counter(int* c, int v) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __hip_atomic_store(c, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Waits until *c >= v, and returns it.  The wavefront waited for is of the same
// workgroup and its own waits are bounded; the limit only makes that plain.
__device__ __forceinline__ int wait_counter(const int* c, int v, int* status) {
  int got = read_counter(c);
#pragma nounroll
  for (int spin = 0; got < v; ++spin) {
    if (spin == (1 << 26)) {
      raise_status(status, kStatusTimeout);
      break;
    }
    __builtin_amdgcn_s_sleep(1);
    got = read_counter(c);
  }
  return got;
}

template <int N, int I = 0, typename F> __device__ __forceinline__ void unroll(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll<N, I + 1>(f);
  }
}

// Bound by the chain of steps: one per level of the triangle, 0.08 to 0.1 us
// each (wavefront 0 issues some 33 instructions a step; the LDS round trip and
// the row's FMAs take 42 ns of it), plus 1 to 2 us per strip that the chain
// crosses; with 13 entries a row by the 10 KB that a step loads: one wavefront
// draws 30 GB/s with 8 loads in flight, 45 with 32, 64 with 56, so those rows'
// records are loaded up to seven steps ahead (strip_fn).  us per triangle, this kernel against a
// wavefront per 64-row box of the grid (waiting once per box) and against a hop
// per level: 128^3 7-point 95 / 165 / 375, 1024^2 9-point 329 / 632 / 2503,
// 128^3 27-point 378 / 485 / 2196, 256 2-D ILU(0) factors 112 / 190 / 561.
//
// Workgroups claim strips from a ticket, in dependency order (by the sum of
// the strips' lane coordinates): whatever a strip reads belongs to strips
// that running workgroups claimed before it, so the grid always progresses,
// however many of its workgroups are resident.
//
// Four wavefronts share a strip.  One counter covers all of a wavefront's loads
// and stores in order, so a wavefront that did everything would wait for its
// stores' and polls' round trips at every step:
//   0 solves: loads the records, D - 1 steps ahead; step s reads its entries
//     from the ring (the last steps of the strip's own lanes and of its ghost
//     lines) and sums them in stored order with FMA; the result goes to the
//     ring, and to xp for the lanes that other strips read;
//   1 brings in the ghost lines: a round of two loads polls the values of
//     several steps, and what has arrived goes into the ring (overlapping two
//     rounds only adds traffic: 128^3 7-point 100 us against 96);
//   2 stores results to the caller's x, eight steps at a time: a line's rows
//     are then neighbours in memory, where one step's are 64 lines apart (and
//     it looks once per eight steps: 1024^2 9-point, whole solve of both
//     triangles repeated, 735 us with a look per step, 691 so, 665 with the
//     solver's own looks at wavefronts 2 and 3 read ahead; 740 where the
//     records come from memory every time);
//   3 loads b the same way, into LDS.
// With A = 4 slot q adds to partial sum q mod 4, and the sums are added in the
// order of the row-wise kernels' butterfly (rows that those kernels give fewer
// lanes leave the upper sums at -0, which changes nothing): the same bits as
// every other schedule.  All loads go to addresses clamped to the line's own
// run instead of under a mask, so that the number in flight is fixed and
// waiting for one step's never waits for a later step's.
//
// Several right-hand sides: a task is one column of one strip, since a strip
// holds up its neighbours by its steps' latency, which more columns per task
// lengthen, while other columns' strips fill the other compute units.  Whole
// solves, us, 128^3 triangle, 16 columns, 1 / 2 / 3 / 4 columns per task:
// 422 / 540 / 513 / 592 (row-wise: 983); ILU(0) 96^3, FP32, 3 columns:
// 76 / 92 / 138 / 135 (332).
constexpr int kStripThreads = 256;
constexpr int kBlock = 8;                    // steps that wavefronts 2 and 3 take at once
constexpr int kBCols = 65;                   // row of the b ring, padded against bank conflicts
static_assert(kBlock == 8, "eight steps of eight cache lines to a wavefront");
constexpr int kXCols = kBlock + 1;           // line of the store scratch, likewise

template <typename T, int E, int A, int D>
__global__ void __launch_bounds__(kStripThreads, 1) k_strip(SArgs<T> a) {
  constexpr int VW = sizeof(T) / 4;
  constexpr int CW = (E + 1) * VW;                     // first word of the ring addresses
  constexpr int NW = CW + (E + 1) / 2;
  constexpr int NQ = NW / 4, NT = NW % 4;
  constexpr unsigned kRowBytes = kRingCols * sizeof(T);
  constexpr unsigned kRingMask = kRingSteps * kRowBytes - sizeof(T);
  static_assert(A == 1 || E % 2 == 1, "the partial-sum count takes the spare half word");
  static_assert(kRingSteps % D == 0 && kRingSteps % kBlock == 0, "stages follow the ring");
  __shared__ __attribute__((aligned(16))) T ring[kRingSteps * kRingCols];
  __shared__ T bring[kRingSteps * kBCols];
  __shared__ T xout[64 * kXCols];
  __shared__ StripCounters cnt;
  const int lane = threadIdx.x & 63, role = wave_uniform(threadIdx.x >> 6);
  for (;;) {
    if (threadIdx.x == 0) cnt.strip = atomicAdd(a.ticket, 1);
    __syncthreads();
    const int task = wave_uniform(cnt.strip);
    if (task >= a.nstrips * a.nrhs) return;            // the whole workgroup
    // several right-hand sides: the columns of a strip follow one another
    const int p = task / a.nrhs, column = task - p * a.nrhs;
    const T* const b = a.b + column * a.ld;
    T* const x = a.x + column * a.ld;
    T* const xp = a.xp + column * a.npub;
    const StripInfo inf = a.info[p];
    const StripLane* lanes = a.lane + static_cast<int64_t>(p) * 64;
    const int steps = wave_uniform(inf.steps), stride = wave_uniform(inf.stride),
              npub = wave_uniform(inf.npub);
    for (int q = threadIdx.x; q < kRingSteps * kRingCols; q += kStripThreads) ring[q] = T(0);
    if (threadIdx.x == 0) cnt.avail = cnt.bready = cnt.done = cnt.stored = 0;
    __syncthreads();
    if (role == 0) {
      const StripLane l = lanes[lane];
      // Steps are clamped to those of the eight lanes that share a cache line:
      // lane by lane, every lane that has ended would add a line of its own to
      // every load (128^3 27-point: 829 us against 415).
      const int rlo = l.rlo, rhi = l.rhi;
      const int64_t rec0 = uniform64(inf.rec0);
      const char* quad = a.quad + rec0 * (NQ * 1024);
      const char* tail = a.tail + rec0 * (NT * 256);
      // lanes that nobody reads publish into a line of the strip's own, so
      // that the store is unconditional and counted like the loads
      T* pub = l.pub >= 0 ? xp + inf.pub0 + l.pub
                          : a.xp + a.npub * a.nrhs + task * static_cast<int64_t>(kDumpSlot) +
                                lane % kDumpSlot;
      const int64_t pub_step = l.pub >= 0 ? npub : 0;
      unsigned w[D][NW];
      auto fetch = [&](auto k, int s) {
        const int sc = min(max(s, rlo), rhi);
        const unsigned oq = __umul24(sc, NQ * 1024) + lane * 16u;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const uint4 v = *reinterpret_cast<const uint4*>(quad + oq + q * 1024);
          w[k][4 * q] = v.x;
          w[k][4 * q + 1] = v.y;
          w[k][4 * q + 2] = v.z;
          w[k][4 * q + 3] = v.w;
        }
        if constexpr (NT > 0) {
          const unsigned ot = __umul24(sc, NT * 256) + lane * (NT * 4u);
          const auto v = *reinterpret_cast<const Words<NT>*>(tail + ot);
#pragma unroll
          for (int q = 0; q < NT; ++q) w[k][4 * NQ + q] = v.w[q];
        }
      };
      // Ring addresses of a step's entries, taken apart one step ahead.
      // Entries only ever name rows that exist (or the zero column), so what
      // lanes without a row at a step compute is never read.
      unsigned at[2][E];
      auto address = [&](auto k, auto h) {
#pragma unroll
        for (int q = 0; q < E; ++q) {
          at[h][q] = (q % 2 ? w[k][CW + q / 2] >> 16 : w[k][CW + q / 2]) & kRingMask;
          asm volatile("" : "+v"(at[h][q]));   // here, not in front of the reads
        }
      };
      int avail = 0;
      auto step = [&](auto kc, int s) {
        constexpr int row = decltype(kc)::value % kRingSteps, k0 = decltype(kc)::value % D;
        constexpr std::integral_constant<int, k0> k{};
        constexpr std::integral_constant<int, (k0 + 1) % D> kn{};
        constexpr std::integral_constant<int, (k0 + D - 1) % D> kp{};
        constexpr std::integral_constant<int, k0 % 2> h{};
        constexpr std::integral_constant<int, (k0 + 1) % 2> hn{};
        if (__builtin_expect(avail < s, 0)) avail = wait_counter(&cnt.avail, s, a.status);
        T g[E];
#pragma unroll
        for (int q = 0; q < E; ++q)
          g[q] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(ring) + at[h][q]);
        const T bi = bring[row * kBCols + lane];
        const int seen = __hip_atomic_load(&cnt.avail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // while the reads are on their way: the stage of the last step is
        // free, and the next step's addresses
        fetch(kp, s + D - 1);
        address(kn, hn);
        T v[E + 1];
        __builtin_memcpy(v, w[k], sizeof(v));
        T sum[A];
        sum[0] = T(0);
        if constexpr (A == 4) {
          const int n = 1 << ((w[k][CW + E / 2] >> 16) & 3);
#pragma unroll
          for (int q = 1; q < A; ++q) sum[q] = q < n ? T(0) : -T(0);
        }
#pragma unroll
        for (int q = 0; q < E; ++q) sum[q % A] = fma_t(v[q], g[q], sum[q % A]);
        T tot = sum[0];
        if constexpr (A == 4) tot = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        const T xi = canonical((bi - tot) * v[E]);
        ring[row * kRingCols + lane] = xi;
        write_counter(&cnt.done, s + 1);
        store_agent(pub, xi);
        pub += pub_step;
        avail = wave_uniform(seen);
      };
      unroll<D - 1>([&](auto k) { fetch(k, k); });
      address(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
      constexpr int U = kRingSteps;
      int bready = 0, stored = 0;
      for (int s = 0; s < steps; s += U)
        unroll<U>([&](auto k) {
          // every eight steps: their b is in place, and the rows that they
          // overwrite have been taken over (both read a step early, so that the
          // solver does not stand still for the LDS)
          if constexpr (k % kBlock == 0) {
            const int b_end = s + k + kBlock, x_end = b_end - kRingSteps;
            if (__builtin_expect(wave_uniform(bready) < b_end, 0))
              wait_counter(&cnt.bready, b_end, a.status);
            if (__builtin_expect(wave_uniform(stored) < x_end, 0))
              wait_counter(&cnt.stored, x_end, a.status);
          }
          if constexpr (k % kBlock == kBlock - 1) {
            bready = __hip_atomic_load(&cnt.bready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            stored = __hip_atomic_load(&cnt.stored, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
          step(k, s + k);
        });
    } else if (role == 1) {
      // lane = (step, ghost line): one load covers 64 >> lg steps, a round two
      // loads
      const int lg = wave_uniform(inf.ghost_lg), per = 64 >> lg;
      if (lg >= 0) {
        const StripLane l = lanes[lane & ((1 << lg) - 1)];
        const int j = lane >> lg, col = 64 + (lane & ((1 << lg) - 1));
        const int glo = l.glo, ghi = l.glo + (l.glen > 0 ? l.glen - 1 : 0);
        const T* gp = xp + l.gpos;
        int next = 0, done = 0, idle = 0;     // first step not brought in yet
        bool lost = false;
        auto issue = [&](T (&v)[2], int base) {
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const int sc = min(max(base + k * per + j, glo), ghi);
            v[k] = load_agent(gp + static_cast<int64_t>(sc) * npub);
          }
        };
        // brings in the steps from `next` on that the round has complete
        auto take = [&](T (&v)[2], int base) {
          unsigned long long miss[2];
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const bool has = static_cast<unsigned>(base + k * per + j - glo) < static_cast<unsigned>(l.glen);
            if (lost && is_sentinel(v[k])) v[k] = __builtin_nan("");
            miss[k] = __ballot(has && is_sentinel(v[k]));
          }
          // (the solver stops a little past `steps`: nothing is brought in there)
          const int upto = min(steps, base + (miss[0]   ? (__ffsll(miss[0]) - 1) >> lg
                                              : miss[1] ? per + ((__ffsll(miss[1]) - 1) >> lg)
                                                        : 2 * per));
          if (upto <= next && next < steps) {
            // nothing new: give up after spin_limit rounds, or once another
            // wavefront has
            if (++idle > a.spin_limit ||
                ((idle & 31) == 31 && (load_status(a.status) & kStatusTimeout))) {
              raise_status(a.status, kStatusTimeout);
              lost = true;
            }
            return;
          }
          idle = 0;
          // a row of the ring is free once the solver is past the farthest
          // step that an entry reaches back from
          constexpr int kAhead = kRingSteps - kStripMaxBack;
          while (next < upto) {
            if (done + kAhead <= next) done = wait_counter(&cnt.done, next + 1 - kAhead, a.status);
            const int end = min(upto, done + kAhead);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const int t = base + k * per + j;
              if (t >= next && t < end && static_cast<unsigned>(t - glo) < static_cast<unsigned>(l.glen))
                ring[(t & (kRingSteps - 1)) * kRingCols + col] = v[k];
            }
            write_counter(&cnt.avail, end);
            next = end;
          }
        };
        T v[2];
        while (next < steps) {
          const int base = next;
          issue(v, base);
          take(v, base);
        }
      }
      write_counter(&cnt.avail, INT32_MAX);   // the solver rounds its steps up
    } else {
      // line li(i) of instruction i, step s0 + (lane mod kBlock)
      constexpr int L = 64 / kBlock;
      int row0[kBlock], lo[kBlock], n[kBlock];
#pragma unroll
      for (int i = 0; i < kBlock; ++i) {
        const StripLane l = lanes[i * L + lane / kBlock];
        row0[i] = l.row0;
        lo[i] = l.lo;
        n[i] = l.len;
      }
      const int j = lane % kBlock;
      if (role == 2) {
        int done = 0;
        for (int s0 = 0; s0 < steps; s0 += kBlock) {
          const int end = min(s0 + kBlock, steps);
          if (done < end) done = wait_counter(&cnt.done, end, a.status);
          T xs[kBlock];
#pragma unroll
          for (int q = 0; q < kBlock; ++q) xs[q] = ring[((s0 + q) & (kRingSteps - 1)) * kRingCols + lane];
#pragma unroll
          for (int q = 0; q < kBlock; ++q) xout[lane * kXCols + q] = xs[q];
          write_counter(&cnt.stored, end);
#pragma unroll
          for (int i = 0; i < kBlock; ++i) {
            const T xi = xout[(i * L + lane / kBlock) * kXCols + j];
            if (static_cast<unsigned>(s0 + j - lo[i]) < static_cast<unsigned>(n[i]))
              x[row0[i] + static_cast<int64_t>(s0 + j) * stride] = xi;
          }
        }
        write_counter(&cnt.stored, INT32_MAX);
      } else {
        constexpr int P = 3;                           // blocks in flight
        T v[P][kBlock];
        auto fetch = [&](auto k, int s0) {
#pragma unroll
          for (int i = 0; i < kBlock; ++i) {
            const int sc = min(max(s0 + j, lo[i]), lo[i] + max(n[i], 1) - 1);
            v[k][i] = b[row0[i] + static_cast<int64_t>(sc) * stride];
          }
        };
        unroll<P>([&](auto k) {
          fetch(k, k * kBlock);
        });
        for (int s = 0; s < steps; s += P * kBlock)
          unroll<P>([&](auto k) {
            const int s0 = s + k * kBlock;
            wait_counter(&cnt.done, s0 + kBlock - kRingSteps, a.status);
#pragma unroll
            for (int i = 0; i < kBlock; ++i)
              bring[((s0 + j) & (kRingSteps - 1)) * kBCols + i * L + lane / kBlock] = v[k][i];
            write_counter(&cnt.bready, s0 + kBlock);
            fetch(k, s0 + P * kBlock);
          });
        write_counter(&cnt.bready, INT32_MAX);
      }
    }
    __syncthreads();                                   // the strip is done
  }
}

// The kernel for a copy.
template <typename T> const void* strip_fn(const DevStrips& t, int nrhs) {
  const int acc = strip_sums(t, nrhs), depth = strip_depth(t, sizeof(T), nrhs);
#define SPTRSV_STRIP(E, A, D)                                \
  if (t.entries == E && acc == A && depth == D)              \
  return reinterpret_cast<const void*>(k_strip<T, E, A, D>)
  SPTRSV_STRIP(2, 1, 16);
  SPTRSV_STRIP(3, 1, 16);
  SPTRSV_STRIP(4, 1, 16);
  SPTRSV_STRIP(13, 4, 8);
  SPTRSV_STRIP(15, 4, 8);
  SPTRSV_STRIP(13, 1, 8);
  SPTRSV_STRIP(15, 1, 8);
  if constexpr (sizeof(T) == 8) {
    SPTRSV_STRIP(13, 4, 4);
    SPTRSV_STRIP(15, 4, 4);
    SPTRSV_STRIP(13, 1, 4);
    SPTRSV_STRIP(15, 1, 4);
  }
#undef SPTRSV_STRIP
  return nullptr;
}

inline int blocks(int64_t work, int per) {
  const int64_t b = (work + per - 1) / per;
  return static_cast<int>(b < 1 ? 1 : b < (1 << 30) ? b : (1 << 30));
}

struct DevFree {
  std::vector<void*> p;
  ~DevFree() {
    for (void* q : p) dev_free(q);
  }
  template <typename T> bool get(T** out, int64_t count) {
    void* q = nullptr;
    if (dev_alloc(&q, count * static_cast<int64_t>(sizeof(T))) != hipSuccess) return false;
    p.push_back(q);
    *out = static_cast<T*>(q);
    return true;
  }
};

}  // namespace

hipError_t launch_strip_offsets(int n, int64_t nnz, const int* row_ptr, const int* col, int nsys,
                                const int* sys_row0, int* table, int* full, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int rows = offset_rows(n, nsys);
  k_strip_offsets<<<blocks(n, rows), 256, 0, s>>>(n, nnz, row_ptr, col, nsys, sys_row0, rows, table,
                                                  full);
  return hipGetLastError();
}

hipError_t launch_strip_lanes(const DevChunks& c, unsigned char* lanes_lg, hipStream_t s) {
  if (c.count == 0) return hipSuccess;
  k_strip_lanes<<<blocks(static_cast<int64_t>(c.count) * 64, 256), 256, 0, s>>>(c.count, c.start,
                                                                               c.meta, lanes_lg);
  return hipGetLastError();
}

template <typename T> hipError_t launch_strip_gather(const DevPlan& p, const DevStrips& t,
                                                     hipStream_t s) {
  if (t.nrec == 0) return hipSuccess;
  k_strip_gather<T><<<blocks(t.nrec * 64, 256), 256, 0, s>>>(
      t, static_cast<const T*>(p.off_val), static_cast<const T*>(p.dinv));
  return hipGetLastError();
}

void free_strips(DevStrips& t) {
  dev_free(t.mem);
  t = DevStrips();
}

int build_strips(const DevPlan& p, const std::vector<StripGrid>& grids, int max_len,
                 const unsigned char* lanes_lg, int vb, hipStream_t s, DevStrips& out) {
  out = DevStrips();
  const int nsys = static_cast<int>(grids.size());
  if (p.n == 0 || nsys == 0 || max_len > kStripMaxEntries || !p.row_pos) return kErrNotSupported;
  int64_t nboxes = 0;
  std::vector<int> box0(nsys + 1);
  std::vector<StripGrid> gh(grids);
  for (int k = 0; k < nsys; ++k) {
    gh[k].box0 = box0[k] = static_cast<int>(nboxes);
    nboxes += gh[k].n > 0 ? static_cast<int64_t>(gh[k].nbu) * gh[k].nbv : 0;
    if (nboxes > (1 << 22)) return kErrNotSupported;
    if ((gh[k].axis == 0 ? gh[k].nx : gh[k].axis == 1 ? gh[k].ny : gh[k].nz) > kStripMaxSteps)
      return kErrNotSupported;
  }
  box0[nsys] = static_cast<int>(nboxes);
  const int acc = lanes_lg ? 4 : 1;
  // One block: uploaded [grids, box0, cnt], downloaded [cnt, box], uploaded again
  // [boxes, box_strip] (allocations, frees and copies are what the set-up of a
  // small triangle takes: 10 to 20 us each in a busy process).
  auto up = [](int64_t b) { return (b + 255) / 256 * 256; };
  const int64_t b_grids = up(nsys * static_cast<int64_t>(sizeof(StripGrid))), b_box0 = up((nsys + 1) * 4ll),
                b_cnt = up(sizeof(StripCount)), b_box = up(nboxes * static_cast<int64_t>(sizeof(int2))),
                b_boxes = up(nboxes * static_cast<int64_t>(sizeof(StripBox))), b_strip = up(nboxes * 4);
  DevFree f;
  char* work = nullptr;
  if (!f.get(&work, b_grids + b_box0 + b_cnt + b_box + b_boxes + b_strip)) return kErrOom;
  StripGrid* const grids_d = reinterpret_cast<StripGrid*>(work);
  int* const box0_d = reinterpret_cast<int*>(work + b_grids);
  StripCount* const cnt = reinterpret_cast<StripCount*>(work + b_grids + b_box0);
  int2* const box_d = reinterpret_cast<int2*>(work + b_grids + b_box0 + b_cnt);
  char* const boxes_at = work + b_grids + b_box0 + b_cnt + b_box;
  StripBox* const boxes_d = reinterpret_cast<StripBox*>(boxes_at);
  int* const box_strip_d = reinterpret_cast<int*>(boxes_at + b_boxes);
  StripCount c{0, 0, 0};
  if (!lanes_lg) c.slots = max_len;   // an entry, a slot
  std::vector<char> host(b_grids + b_box0 + b_cnt);
  std::memcpy(host.data(), gh.data(), nsys * sizeof(StripGrid));
  std::memcpy(host.data() + b_grids, box0.data(), (nsys + 1) * sizeof(int));
  std::memcpy(host.data() + b_grids + b_box0, &c, sizeof(c));
#define TCHK(expr)                            \
  do {                                        \
    if ((expr) != hipSuccess) return kErrHip; \
  } while (0)
  TCHK(hipMemcpyAsync(work, host.data(), host.size(), hipMemcpyHostToDevice, s));
  if (lanes_lg) {
    k_strip_slots<<<std::min(blocks(p.n, 256), 1024), 256, 0, s>>>(p.n, p.off_ptr, lanes_lg, cnt);
    TCHK(hipGetLastError());
  }
  k_strip_boxes<<<static_cast<int>(nboxes), 64, 0, s>>>(grids_d, nsys, box0_d, box_d, cnt);
  TCHK(hipGetLastError());
  std::vector<char> found(b_cnt + nboxes * sizeof(int2));
  TCHK(hipMemcpyAsync(found.data(), cnt, found.size(), hipMemcpyDeviceToHost, s));
  TCHK(hipStreamSynchronize(s));
  std::memcpy(&c, found.data(), sizeof(c));
  std::vector<int2> box(nboxes);
  std::memcpy(box.data(), found.data() + b_cnt, nboxes * sizeof(int2));
  DevStrips t;
  t.acc = acc;
  t.entries = acc == 1 ? std::max(2, c.slots) : c.slots <= 13 ? 13 : 15;
  if (c.slots > (acc == 1 ? 4 : 15) || c.rows != static_cast<unsigned long long>(p.n))
    return kErrNotSupported;
  // strips in dependency order: by the sum of the lane coordinates, so that
  // whatever a strip reads is earlier
  std::vector<StripBox> boxes;
  std::vector<int> order;
  {
    std::vector<StripBox> all;
    std::vector<int> id;
    int last = 0;
    for (int k = 0; k < nsys; ++k)
      for (int q = 0; gh[k].n > 0 && q < gh[k].nbu * gh[k].nbv; ++q)
        if (box[gh[k].box0 + q].y > 0) {
          all.push_back(StripBox{k, q % gh[k].nbu, q / gh[k].nbu, box[gh[k].box0 + q].x});
          id.push_back(gh[k].box0 + q);
          last = std::max(last, all.back().bu + all.back().bv);
        }
    std::vector<int> at(last + 2, 0);
    for (const StripBox& b : all) at[b.bu + b.bv + 1]++;
    for (int q = 0; q <= last; ++q) at[q + 1] += at[q];
    boxes.resize(all.size());
    order.resize(all.size());
    for (size_t q = 0; q < all.size(); ++q) {
      const int w = at[all[q].bu + all[q].bv]++;
      boxes[w] = all[q];
      order[w] = id[q];
    }
  }
  t.nstrips = static_cast<int>(boxes.size());
  std::vector<StripInfo> info(t.nstrips);
  std::vector<int> box_strip(nboxes, -1);
  int max_steps = 0;
  for (int q = 0; q < t.nstrips; ++q) {
    const StripGrid& g = gh[boxes[q].sys];
    const int steps = box[order[q]].y;
    int lg = -1;
    if (g.nghost > 0)
      for (lg = 0; (1 << lg) < g.nghost;) ++lg;
    info[q] = StripInfo{steps, g.stride, g.npub, boxes[q].bu + boxes[q].bv > 0 ? lg : -1, t.nrec, t.npub};
    box_strip[order[q]] = q;
    t.nrec += steps;
    // the solver rounds its steps up to the ring's and publishes in all of them
    t.npub += static_cast<int64_t>((steps + kRingSteps - 1) / kRingSteps * kRingSteps) * g.npub;
    max_steps = std::max(max_steps, steps);
  }
  // lanes without a row cost memory: grids far from the strips' shape keep
  // the row-wise schedules (batches of 16x16 grids, eight lanes a row, are
  // still faster in strips); the gather has a thread per lane
  if (t.nstrips == 0 || t.nrec * 64 > 16ll * p.n + (1 << 20) || t.nrec * 64 > UINT32_MAX || max_steps > kStripMaxSteps)
    return kErrNotSupported;
  const int E = t.entries, vw = vb / 4;
  t.words = (E + 1) * vw + (E + 1) / 2;
  const int nq = t.words / 4, nt = t.words % 4;
  const int64_t b_quad = up(t.nrec * nq * 1024), b_tail = up(t.nrec * nt * 256),
                b_src = up(t.nrec * E * 256), b_dsrc = up(t.nrec * 256),
                b_lane = up(t.nstrips * 64ll * sizeof(StripLane)),
                b_info = up(t.nstrips * static_cast<int64_t>(sizeof(StripInfo)));
  if (dev_alloc(&t.mem, b_quad + b_tail + b_src + b_dsrc + b_lane + b_info) != hipSuccess)
    return kErrOom;
  char* at = static_cast<char*>(t.mem);
  auto take = [&](int64_t b) {
    char* q = at;
    at += b;
    return q;
  };
  t.quad = take(b_quad);
  t.tail = reinterpret_cast<unsigned*>(take(b_tail));
  t.src = reinterpret_cast<int*>(take(b_src));
  t.dsrc = reinterpret_cast<int*>(take(b_dsrc));
  t.lane = reinterpret_cast<StripLane*>(take(b_lane));
  t.info = reinterpret_cast<StripInfo*>(take(b_info));
  hipError_t e = hipMemcpyAsync(t.info, info.data(), info.size() * sizeof(StripInfo),
                                hipMemcpyHostToDevice, s);
  std::vector<char> order_h(b_boxes + nboxes * sizeof(int));
  std::memcpy(order_h.data(), boxes.data(), boxes.size() * sizeof(StripBox));
  std::memcpy(order_h.data() + b_boxes, box_strip.data(), nboxes * sizeof(int));
  if (e == hipSuccess)
    e = hipMemcpyAsync(boxes_at, order_h.data(), order_h.size(), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) {
    k_strip_lanes_of<<<t.nstrips, 64, 0, s>>>(grids_d, boxes_d, box_strip_d, t, cnt);
    const unsigned y = record_blocks(t.nrec, t.nstrips, max_steps);
    auto* const fn = y * kRecordWaves < static_cast<unsigned>(max_steps) ? k_strip_records<true>
                                                                         : k_strip_records<false>;
    fn<<<dim3(t.nstrips, y), kRecordThreads, 0, s>>>(p.off_ptr, p.off_col, p.row_pos, lanes_lg,
                                                     grids_d, boxes_d, vb, t, cnt);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&c, cnt, sizeof(c), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess || c.bad) {
    free_strips(t);
    return e != hipSuccess ? kErrHip : kErrNotSupported;
  }
#undef TCHK
  out = t;
  return kOk;
}

template <typename T> hipError_t launch_strip_solve(const StripSolveArgs& sa, hipStream_t s) {
  const DevStrips& t = *sa.strips;
  if (t.nstrips == 0) return hipSuccess;
  SArgs<T> a;
  a.nstrips = t.nstrips;
  a.nrhs = sa.nrhs;
  a.ld = sa.ld;
  a.npub = t.npub;
  a.info = t.info;
  a.lane = t.lane;
  a.quad = static_cast<const char*>(t.quad);
  a.tail = reinterpret_cast<const char*>(t.tail);
  a.b = static_cast<const T*>(sa.b);
  a.x = static_cast<T*>(sa.x);
  a.xp = static_cast<T*>(sa.xp);
  a.status = sa.scratch.status;
  a.ticket = sa.scratch.arrive;
  a.spin_limit = sa.spin_limit;
  const void* fn = strip_fn<T>(t, sa.nrhs);
  if (!fn) return hipErrorInvalidValue;
  void* args[] = {&a};
  return hipLaunchKernel(fn, dim3(sa.grid), dim3(kStripThreads), args, 0, s);
}

template <typename T> int strip_blocks_per_cu(const DevStrips& t, int nrhs) {
  const void* fn = strip_fn<T>(t, nrhs);
  int nb = 0;
  if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, kStripThreads, 0) != hipSuccess) return 1;
  return nb > 0 ? nb : 1;
}

#define SPTRSV_INSTANTIATE(T)                                                                 \
  template hipError_t launch_strip_gather<T>(const DevPlan&, const DevStrips&, hipStream_t);  \
  template hipError_t launch_strip_solve<T>(const StripSolveArgs&, hipStream_t);              \
  template int strip_blocks_per_cu<T>(const DevStrips&, int);

SPTRSV_INSTANTIATE(double)
SPTRSV_INSTANTIATE(float)

}  // namespace sptrsv
