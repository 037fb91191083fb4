// Device-side setup phase: validity check, levels, level-ordered layout.
// Section references are to Li, arXiv:1710.04985.
#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include <algorithm>

#include "analysis.hpp"
#include "analysis_gpu.hpp"
#include "device_common.hpp"
#include "devmem.hpp"

namespace sptrsv {
namespace {

enum : int { kFlagBad = 1, kFlagUnsorted = 2, kFlagTimeout = 4 };

__device__ __forceinline__ int bitlen(unsigned v) { return v ? 32 - __builtin_clz(v) : 0; }

// Raises *out to the largest v of the workgroup (256 threads, all of them):
// one atomic per workgroup at most, and none that would change nothing.
__device__ __forceinline__ void block_max(int v, int* out) {
  __shared__ int wave[4];
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  if ((threadIdx.x & 63) == 0) wave[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    v = max(max(wave[0], wave[1]), max(wave[2], wave[3]));
    if (v > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(out, v);
  }
}

// One row per thread: bounds, column range and side, strictly increasing
// columns, one diagonal (unless unit), dependency count.  Any irregularity
// only raises a flag; the host analysis then decides the exact error.
__global__ void __launch_bounds__(256) k_check(int n, int64_t nnz, const int* __restrict__ rp,
                                               const int* __restrict__ col, int upper, int unit,
                                               int* __restrict__ depcnt, int* flags, int* maxlen) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  int f = 0, ml = 0;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < n; t += stride) {
    const int i = static_cast<int>(t);
    const int a = rp[i], b = rp[i + 1];
    depcnt[i] = 0;
    if (a < 0 || b < a || b > nnz) {
      f |= kFlagBad;
      continue;
    }
    int nd = 0, dep = 0, prev = -1;
    for (int e = a; e < b; ++e) {
      const int j = col[e];
      if (j < 0 || j >= n) {
        f |= kFlagBad;
        break;
      }
      if (upper ? j < i : j > i) f |= kFlagBad;
      if (e > a && j <= prev) f |= kFlagUnsorted;
      prev = j;
      if (j == i) ++nd;
      else ++dep;
    }
    if (nd > 1 || (!unit && nd != 1)) f |= kFlagBad;
    depcnt[i] = dep;
    ml = dep > ml ? dep : ml;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && (rp[0] != 0 || rp[n] != nnz)) f |= kFlagBad;
  if (f) atomicOr(flags, f);
  block_max(ml, maxlen);
}

__global__ void __launch_bounds__(256) k_fill_int(int* p, int64_t count, int v) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < count; t += stride)
    p[t] = v;
}

// Levels of rows on grids without gaps: each row is given the level that its
// place in the grid calls for, and checked against its dependencies, which
// are given theirs the same way.  The recurrence has one solution, so levels
// that satisfy it at every row are the levels; otherwise *differ is set and
// nothing else here counts.  Bound by the pattern's bytes (128^3 7-point:
// 30 us; the sweep k_levels 2550 us, a hop per level).
__global__ void __launch_bounds__(256)
k_grid_levels(int n, const int* __restrict__ rp, const int* __restrict__ col,
              const StripGrid* __restrict__ grids, int nsys, int* __restrict__ level, int* differ,
              int* maxlev) {
  const int stride = gridDim.x * blockDim.x;
  int top = -1;
  bool bad = false;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < n; t += stride) {
    const int i = static_cast<int>(t);
    int lo = 0, hi = nsys - 1;             // the last system with row0 <= i
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (grids[mid].row0 <= i) lo = mid;
      else hi = mid - 1;
    }
    const StripGrid& g = grids[lo];
    const int want = strip_level(g, i - g.row0);
    int got = 0;
    for (int e = rp[i], e1 = rp[i + 1]; e < e1; ++e) {
      const int j = col[e];
      if (j != i) got = max(got, strip_level(g, j - g.row0) + 1);
    }
    bad |= got != want;
    level[i] = want;
    top = max(top, want);
  }
  if (bad) __hip_atomic_store(differ, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  block_max(top, maxlev);
}

// Levels of Sec. 4.1 (0-based), computed without global synchronisation: the
// self-scheduled sweep with max(level)+1 in place of the dot product.  Rows
// are taken in dependency order (ascending for lower, descending for upper)
// in chunks of 64, one row per lane; each workgroup (one wavefront) claims
// the next chunk from a ticket, so chunks are taken in order by running
// wavefronts and no co-residency is assumed.
// level[] starts at -1; a row publishes its level with one agent-scope atomic
// store.  Rows are sorted on this route, so a row's dependencies inside the
// chunk are the off-diagonals next to its diagonal and those in earlier
// chunks one contiguous range.  A round polls the earlier-chunk range
// (sixteen loads in flight, resuming at the first one not yet published),
// then resolves the chain inside the chunk through LDS, one link per step.
// A lane keeps up to kInChunk in-chunk dependencies (6-bit lane numbers)
// packed in a register and rescans its in-chunk range otherwise.  The lowest
// unfinished row always has every dependency published and its chunk held by
// a running wavefront, so the sweep progresses.
constexpr int kInChunk = 10;

__global__ void __launch_bounds__(64)
k_levels(int n, const int* __restrict__ rp, const int* __restrict__ col, int upper,
         int* level, int* flags, int* maxlev, int* ticket, int spin_limit) {
  __shared__ int sl[64];
  const int lane = threadIdx.x;
  const int nch = (n + 63) / 64;
  int wmax = -1;
  for (;;) {
    int c = 0;
    if (lane == 0) c = atomicAdd(ticket, 1);
    c = __builtin_amdgcn_readfirstlane(c);
    if (c >= nch) break;
    const int c0 = c * 64;            // dependency-order index of lane 0
    const int r = c0 + lane;
    const bool live = r < n;
    const int i = live ? (upper ? n - 1 - r : r) : 0;
    const int a = live ? rp[i] : 0, e1 = live ? rp[i + 1] : 0;
    // Rows are sorted on this route (k_check): the in-chunk dependencies are
    // the off-diagonals next to the diagonal, those in earlier chunks the
    // contiguous range [oa, ob)
    unsigned long long pk = 0;
    int nin = 0, oa = a, ob = a, ib = a, ie = a;
    if (live) {
      if (!upper) {
        int e = e1;
        if (e > a && col[e - 1] == i) --e;          // diagonal last
        ie = e;
        while (e > a && col[e - 1] >= c0) {         // in-chunk: c0 <= j < i
          if (nin < kInChunk) pk |= static_cast<unsigned long long>(col[e - 1] - c0) << (6 * nin);
          ++nin;
          --e;
        }
        ib = e;
        oa = a;
        ob = e;
      } else {
        int e = a;
        if (e < e1 && col[e] == i) ++e;             // diagonal first
        ib = e;
        const int jmax = n - 1 - c0;                // in-chunk: i < j <= n-1-c0
        while (e < e1 && col[e] <= jmax) {
          if (nin < kInChunk)
            pk |= static_cast<unsigned long long>(n - 1 - col[e] - c0) << (6 * nin);
          ++nin;
          ++e;
        }
        ie = e;
        oa = e;
        ob = e1;
      }
    }
    int e = oa;                       // cursor over the earlier-chunk dependencies
    int lvl = 0;
    bool done = !live;
    sl[lane] = -1;
    for (int round = 0;; ++round) {
      bool gready = true;
      if (!done) {
        // sixteen at a time: their columns, then their levels, in flight together
        while (e < ob) {
          int v16[16];
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            const int j = e + q < ob ? col[e + q] : -1;
            v16[q] = j >= 0 ? __hip_atomic_load(level + j, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT)
                            : 0;
          }
          int adv = 0;
          bool stop = false;
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            if (stop || e + q >= ob) continue;
            if (v16[q] < 0) {
              stop = true;
            } else {
              lvl = v16[q] + 1 > lvl ? v16[q] + 1 : lvl;
              ++adv;
            }
          }
          e += adv;
          if (stop) {
            gready = false;
            break;
          }
        }
      }
      for (int step = 0; step < 65; ++step) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        bool progressed = false;
        if (!done && gready) {
          int l2 = lvl;
          bool ready = true;
          if (nin <= kInChunk) {
            for (int q = 0; q < nin; ++q) {
              const int v = sl[(pk >> (6 * q)) & 63];
              if (v < 0) {
                ready = false;
                break;
              }
              l2 = v + 1 > l2 ? v + 1 : l2;
            }
          } else {
            for (int e2 = ib; e2 < ie; ++e2) {
              const int rj = upper ? n - 1 - col[e2] : col[e2];
              const int v = sl[rj - c0];
              if (v < 0) {
                ready = false;
                break;
              }
              l2 = v + 1 > l2 ? v + 1 : l2;
            }
          }
          if (ready) {
            __hip_atomic_store(level + i, l2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sl[lane] = l2;
            wmax = l2 > wmax ? l2 : wmax;
            done = true;
            progressed = true;
          }
        }
        if (!__any(progressed)) break;
      }
      if (__all(done)) break;
      if (round >= spin_limit) {     // cannot happen on a valid triangle: drain
        if (!done) {
          __hip_atomic_store(level + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          done = true;
        }
        if (lane == 0) atomicOr(flags, kFlagTimeout);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const int v = __shfl_xor(wmax, o, 64);
    wmax = v > wmax ? v : wmax;
  }
  if (lane == 0 && wmax >= 0) atomicMax(maxlev, wmax);
}

// sort keys: (level, bit length of the dependency count), values: row
constexpr int kClassBits = 5;

template <typename K>
__global__ void __launch_bounds__(256) k_keys(int n, const int* __restrict__ level,
                                              const int* __restrict__ depcnt, K* __restrict__ key,
                                              int* __restrict__ rows) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < n; t += stride) {
    const int i = static_cast<int>(t);
    key[i] = (static_cast<K>(level[i]) << kClassBits) | bitlen(static_cast<unsigned>(depcnt[i]));
    rows[i] = i;
  }
}

// Workgroups of the kernels that add up over all rows: each ends with an atomic
// on one word, about 10 ns apart, unless it would change nothing.  The check has
// more of them, so that no thread has several long rows (us at 1024 / 4096 /
// 16384: power-law 1M rows 934 / 615 / 611, 128^3 7-point 22 / 18 / 23, 27-point
// 63 / 69 / 67).
constexpr int kCheckBlocks = 4096, kGridLevelBlocks = 1024;

// inverse permutation, row length per position, level pointers
__global__ void __launch_bounds__(256) k_positions(int n, int nlev, const int* __restrict__ pos_row,
                                                   const int* __restrict__ level,
                                                   const int* __restrict__ depcnt,
                                                   int* __restrict__ pos_of, int* __restrict__ cnt,
                                                   int* __restrict__ ilev) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t <= n; t += stride) {
    const int k = static_cast<int>(t);
    if (k == n) {
      cnt[n] = 0;
      ilev[nlev] = n;
      continue;
    }
    const int i = pos_row[k];
    pos_of[i] = k;
    cnt[k] = depcnt[i];
    const int lk = level[i];
    if (k == 0 || level[pos_row[k - 1]] != lk) ilev[lk] = k;
  }
}

// off-diagonal entries of each position, in stored order
__global__ void __launch_bounds__(256) k_offdiag(int n, int unit, const int* __restrict__ rp,
                                                 const int* __restrict__ col,
                                                 const int* __restrict__ pos_row,
                                                 const int* __restrict__ pos_of,
                                                 const int* __restrict__ off_ptr,
                                                 int* __restrict__ off_col, int* __restrict__ off_pos,
                                                 int* __restrict__ off_src, int* __restrict__ diag_src) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < n; t += stride) {
    const int k = static_cast<int>(t);
    const int i = pos_row[k];
    int o = off_ptr[k];
    int ds = -1;
    for (int e = rp[i]; e < rp[i + 1]; ++e) {
      const int j = col[e];
      if (j == i) {
        if (!unit) ds = e;
        continue;
      }
      off_col[o] = j;
      off_pos[o] = pos_of[j];
      off_src[o] = e;
      ++o;
    }
    diag_src[k] = ds;
  }
}

// Entries one level up, and lanes, of every `step`-th position (see near_step):
// counts[0], counts[1]; counts[2]: all entries.  Sixteen lanes per position, since
// some rows are very long (with a thread each, 50,000 rows of a power-law triangle
// took 0.4 ms), and few workgroups, since each ends with two atomics.
constexpr int kNearLanes = 16;

__global__ void __launch_bounds__(256)
k_near(int n, int step, const int* __restrict__ pos_row, const int* __restrict__ level,
       const int* __restrict__ off_ptr, const int* __restrict__ off_col, int* counts) {
  __shared__ int wave[2][4];
  const int lane = threadIdx.x % kNearLanes;
  const int64_t k = static_cast<int64_t>(blockIdx.x * (256 / kNearLanes) + threadIdx.x / kNearLanes) * step;
  int near = 0, lanes = 0;
  if (k < n) {
    const int lev = level[pos_row[k]], e0 = off_ptr[k], e1 = off_ptr[k + 1];
    for (int e = e0 + lane; e < min(e1, e0 + kNearEntries); e += kNearLanes)
      near += level[off_col[e]] == lev - 1;
    if (lane == 0) lanes = default_lanes(e1 - e0);
  }
  for (int o = 32; o > 0; o >>= 1) {
    near += __shfl_xor(near, o, 64);
    lanes += __shfl_xor(lanes, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    wave[0][threadIdx.x >> 6] = near;
    wave[1][threadIdx.x >> 6] = lanes;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int* w = wave[threadIdx.x];
    atomicAdd(counts + threadIdx.x, w[0] + w[1] + w[2] + w[3]);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) counts[2] = off_ptr[n];
}

inline int blocks(int64_t work) {
  int64_t b = (work + 255) / 256;
  if (b < 1) b = 1;
  return static_cast<int>(b < 65536 ? b : 65536);
}

template <typename T> int dmalloc(T** p, int64_t count) {
  *p = nullptr;
  if (dev_alloc(reinterpret_cast<void**>(p), count * static_cast<int64_t>(sizeof(T))) != hipSuccess)
    return kErrOom;
  return kOk;
}

struct Temps {
  int* flags = nullptr;      // and the counters behind it
  StripGrid* grids = nullptr;
  char* work = nullptr;      // only if the caller's spare part is too small
  ~Temps() {
    for (void* p : {static_cast<void*>(flags), static_cast<void*>(grids), static_cast<void*>(work)})
      dev_free(p);
  }
};

__global__ void __launch_bounds__(256) k_fill_iota(int* p, int64_t count) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < count; t += stride)
    p[t] = static_cast<int>(t);
}

// row_of[e] = the row of entry e
__global__ void __launch_bounds__(256) k_row_of(int n, const int* __restrict__ rp,
                                                int* __restrict__ row_of) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < n; t += stride) {
    const int i = static_cast<int>(t);
    for (int e = rp[i]; e < rp[i + 1]; ++e) row_of[e] = i;
  }
}

// entries of T^T (sorted by (column of T, entry)): column = row of T, source
// = entry of T; row pointers of T^T from the first entry of each column
__global__ void __launch_bounds__(256) k_transpose_fill(int n, int64_t nnz,
                                                        const int* __restrict__ col_sorted,
                                                        const int* __restrict__ src_sorted,
                                                        const int* __restrict__ row_of,
                                                        int* __restrict__ colT, int* __restrict__ rpT) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < nnz; t += stride) {
    colT[t] = row_of[src_sorted[t]];
    // the first entry of column c (and of every empty column before it)
    const int c = col_sorted[t];
    const int cprev = t > 0 ? col_sorted[t - 1] : -1;
    for (int j = cprev + 1; j <= c; ++j) rpT[j] = static_cast<int>(t);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const int clast = nnz > 0 ? col_sorted[nnz - 1] : -1;
    for (int j = clast + 1; j <= n; ++j) rpT[j] = static_cast<int>(nnz);
  }
}

// loc[e] = where entry e of the caller's T sits in the forward plan's value
// buffer (off-diagonals, then the diagonal)
__global__ void __launch_bounds__(256) k_value_loc(int n, int64_t noff, const int* __restrict__ off_src,
                                                   const int* __restrict__ diag_src,
                                                   int* __restrict__ loc) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const int64_t total = noff > n ? noff : n;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < total; t += stride) {
    if (t < noff) loc[off_src[t]] = static_cast<int>(t);
    if (t < n && diag_src[t] >= 0) loc[diag_src[t]] = static_cast<int>(noff + t);
  }
}

// value sources of the T^T plan: entries of T^T -> entries of T -> value
// buffer of the forward plan
__global__ void __launch_bounds__(256) k_compose_src(int n, int64_t noff, const int* __restrict__ srcT,
                                                     const int* __restrict__ loc,
                                                     int* __restrict__ off_src,
                                                     int* __restrict__ diag_src) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const int64_t total = noff > n ? noff : n;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < total; t += stride) {
    if (t < noff) off_src[t] = loc[srcT[off_src[t]]];
    if (t < n && diag_src[t] >= 0) diag_src[t] = loc[srcT[diag_src[t]]];
  }
}

// block-diagonal concatenation of `count` systems (one row of the grid per
// system): row pointers and columns shifted by the systems before, values
// copied; a column outside its own system, or row pointers that do not run
// from 0 to the system's nnz, raise the flag
struct SysDesc {
  const int* rp;
  const int* col;
  const void* vals;
  int n;
  int nnz;
  int roff;
  int eoff;
};

__global__ void __launch_bounds__(256) k_concat(const SysDesc* __restrict__ sys, int vb,
                                                int* __restrict__ rp_cat, int* __restrict__ col_cat,
                                                unsigned char* __restrict__ vals_cat, int* flags) {
  const SysDesc d = sys[blockIdx.y];
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  int f = 0;
  const int64_t total = d.nnz > d.n ? d.nnz : d.n;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < total; t += stride) {
    if (t < d.n) rp_cat[d.roff + t] = d.rp[t] + d.eoff;
    if (t < d.nnz) {
      const int j = d.col[t];
      if (j < 0 || j >= d.n) f = 1;
      col_cat[d.eoff + t] = j + d.roff;
      if (vb == 8)
        reinterpret_cast<unsigned long long*>(vals_cat)[d.eoff + t] =
            static_cast<const unsigned long long*>(d.vals)[t];
      else
        reinterpret_cast<unsigned*>(vals_cat)[d.eoff + t] = static_cast<const unsigned*>(d.vals)[t];
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && (d.rp[0] != 0 || d.rp[d.n] != d.nnz)) f = 1;
  if (f) atomicOr(flags, 1);
}

}  // namespace

void free_device_analysis(DeviceAnalysis& a) {
  dev_free(a.mem.base);
  a = DeviceAnalysis();
}

#define DCHK(expr)                                  \
  do {                                              \
    if ((expr) != hipSuccess) {                     \
      free_device_analysis(out);                    \
      return kErrHip;                               \
    }                                               \
  } while (0)
#define DALLOC(ptr, count)                          \
  do {                                              \
    if (dmalloc(&(ptr), (count)) != kOk) {          \
      free_device_analysis(out);                    \
      return kErrOom;                               \
    }                                               \
  } while (0)

namespace {

// Rows ordered by (level, class) into pos_row and by level into jlev, both
// stably: radix sorts of the same keys with and without the class bits.
// work == nullptr: only sets *bytes.
template <typename K>
hipError_t sort_rows(int n, int lev_bits, DeviceAnalysis& out, char* work, int64_t* bytes,
                     hipStream_t s) {
  const int64_t kb = block_bytes(static_cast<int64_t>(n) * sizeof(K));
  K* key = reinterpret_cast<K*>(work);
  K* key_s = reinterpret_cast<K*>(work + kb);
  int* rows = reinterpret_cast<int*>(work + 2 * kb);
  const int64_t rb = block_bytes(static_cast<int64_t>(n) * sizeof(int));
  void* tmp = work ? work + 2 * kb + rb : nullptr;
  const unsigned un = static_cast<unsigned>(n);
  const int end = kClassBits + lev_bits;
  size_t b1 = 0, b2 = 0;
  if (work) {
    k_keys<K><<<blocks(n), 256, 0, s>>>(n, out.level, out.depcnt, key, rows);
    if (const hipError_t e = hipGetLastError()) return e;
    b1 = b2 = static_cast<size_t>(*bytes - (2 * kb + rb));
  }
  hipError_t e = rocprim::radix_sort_pairs(tmp, b1, key, key_s, rows, out.pos_row, un, 0, end, s);
  if (e == hipSuccess)
    e = rocprim::radix_sort_pairs(tmp, b2, key, key_s, rows, out.jlev, un, kClassBits, end, s);
  if (!work) *bytes = 2 * kb + rb + block_bytes(static_cast<int64_t>(std::max(b1, b2)));
  return e;
}

}  // namespace

int device_analysis(int n, int64_t nnz, const int* row_ptr, const int* col, bool upper,
                    bool unit_diag, int num_cu,
                    const std::vector<std::vector<StripGrid>>& guesses, int64_t spare,
                    hipStream_t s, DeviceAnalysis& out) {
  out = DeviceAnalysis();
  if (n < 1 || nnz < 0 || nnz > INT32_MAX || n > (1 << 30)) return kErrNotSupported;
  out.n = n;
  Temps tp;
  {
    // off-diagonals: all entries but the diagonal's (a unit triangle may store any part of it)
    const int64_t noff = unit_diag ? nnz : std::max<int64_t>(0, nnz - n);
    const int64_t nb = block_bytes((static_cast<int64_t>(n) + 1) * sizeof(int));
    const int64_t ob = block_bytes(std::max<int64_t>(1, noff) * sizeof(int));
    out.mem.bytes = 7 * nb + 3 * ob + block_bytes(spare);
    if (dev_alloc(reinterpret_cast<void**>(&out.mem.base), out.mem.bytes) != hipSuccess) {
      out.mem = DevBlock();
      return kErrOom;
    }
    char* at = out.mem.base;
    for (int** p : {&out.level, &out.depcnt, &out.jlev, &out.pos_row, &out.row_pos, &out.diag_src,
                    &out.off_ptr}) {
      *p = reinterpret_cast<int*>(at);
      at += nb;
    }
    for (int** p : {&out.off_col, &out.off_pos, &out.off_src}) {
      *p = reinterpret_cast<int*>(at);
      at += ob;
    }
    out.spare = at;
  }
  // [0] flags, [1] max row length, [2] max level, [3] chunk ticket, [4] grid levels
  // differ, [5] to [7] k_near's counts
  DALLOC(tp.flags, 8);
  const int init[8] = {0, 0, -1, 0, 0, 0, 0, 0};
  int got[8] = {0, 0, -1, 0, 1, 0, 0, 0};
  DCHK(hipMemcpyAsync(tp.flags, init, sizeof(init), hipMemcpyHostToDevice, s));
  k_check<<<std::min(blocks(n), kCheckBlocks), 256, 0, s>>>(n, nnz, row_ptr, col, upper, unit_diag,
                                                            out.depcnt, tp.flags, tp.flags + 1);
  DCHK(hipGetLastError());
  DCHK(hipMemcpyAsync(got, tp.flags, 2 * sizeof(int), hipMemcpyDeviceToHost, s));
  DCHK(hipStreamSynchronize(s));
  if (got[0]) {
    free_device_analysis(out);
    return kErrNotSupported;
  }
  const int max_len = got[1];

  // levels: from the grid, if a guess of it holds, else by the sweep
  for (const std::vector<StripGrid>& g : guesses) {
    if (!tp.grids) DALLOC(tp.grids, static_cast<int64_t>(g.size()));
    DCHK(hipMemcpyAsync(tp.grids, g.data(), g.size() * sizeof(StripGrid), hipMemcpyHostToDevice, s));
    DCHK(hipMemcpyAsync(tp.flags + 2, init + 2, 3 * sizeof(int), hipMemcpyHostToDevice, s));
    k_grid_levels<<<std::min(blocks(n), kGridLevelBlocks), 256, 0, s>>>(
        n, row_ptr, col, tp.grids, static_cast<int>(g.size()), out.level, tp.flags + 4,
        tp.flags + 2);
    DCHK(hipGetLastError());
    DCHK(hipMemcpyAsync(got, tp.flags, sizeof(got), hipMemcpyDeviceToHost, s));
    DCHK(hipStreamSynchronize(s));
    if (!got[4]) break;
  }
  if (got[4]) {
    got[4] = 1;
    DCHK(hipMemcpyAsync(tp.flags + 2, init + 2, 3 * sizeof(int), hipMemcpyHostToDevice, s));
    k_fill_int<<<blocks(n), 256, 0, s>>>(out.level, n, -1);
    DCHK(hipGetLastError());
    int per_cu = 0;
    DCHK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_levels, 64, 0));
    const int nch = (n + 63) / 64;
    // A waiting lane rereads up to sixteen dependencies per round, so rows
    // longer than that multiply the polling traffic of every wavefront that
    // waits ahead of the level front.  With such rows four wavefronts per CU
    // are used (random power-law triangle: 24 -> 14 ms), otherwise every
    // resident one (mesh triangles, whose level front spans all rows: 6.8 ms,
    // 12.6 ms at four per CU).
    const int waves_per_cu = max_len > 16 ? std::min(4, std::max(1, per_cu)) : std::max(1, per_cu);
    const int grid = std::max(1, std::min(nch, waves_per_cu * num_cu));
    k_levels<<<grid, 64, 0, s>>>(n, row_ptr, col, upper ? 1 : 0, out.level, tp.flags,
                                 tp.flags + 2, tp.flags + 3, 1 << 24);
    DCHK(hipGetLastError());
    DCHK(hipMemcpyAsync(got, tp.flags, 3 * sizeof(int), hipMemcpyDeviceToHost, s));
    DCHK(hipStreamSynchronize(s));
    if (got[0] & kFlagTimeout) {
      free_device_analysis(out);
      return kErrTimeout;
    }
  }
  out.max_row_len = max_len;
  out.nlev = got[2] + 1;
  const int nlev = out.nlev;
  int lev_bits = 1;
  while (lev_bits < 31 && (1ll << lev_bits) < nlev) ++lev_bits;

  // work space: row lengths by position, level pointers, sort and scan buffers
  const bool wide = kClassBits + lev_bits > 32;
  const int64_t cb = block_bytes((static_cast<int64_t>(n) + 1) * sizeof(int));
  const int64_t lb = block_bytes((static_cast<int64_t>(nlev) + 1) * sizeof(int));
  int64_t sort_bytes = 0;
  size_t scan_bytes = 0;
  DCHK(wide ? sort_rows<unsigned long long>(n, lev_bits, out, nullptr, &sort_bytes, s)
            : sort_rows<unsigned>(n, lev_bits, out, nullptr, &sort_bytes, s));
  DCHK(rocprim::exclusive_scan(nullptr, scan_bytes, static_cast<int*>(nullptr), out.off_ptr, 0,
                               static_cast<size_t>(n) + 1, rocprim::plus<int>(), s));
  const int64_t need = cb + lb + std::max(sort_bytes, static_cast<int64_t>(scan_bytes));
  char* work = out.spare;
  if (need > spare) {
    DALLOC(tp.work, need);
    work = tp.work;
  }
  int* cnt = reinterpret_cast<int*>(work);
  int* ilev = reinterpret_cast<int*>(work + cb);
  char* tmp = work + cb + lb;
  DCHK(wide ? sort_rows<unsigned long long>(n, lev_bits, out, tmp, &sort_bytes, s)
            : sort_rows<unsigned>(n, lev_bits, out, tmp, &sort_bytes, s));

  // inverse permutation, row lengths, level pointers, CSR pointers
  k_positions<<<blocks(static_cast<int64_t>(n) + 1), 256, 0, s>>>(n, nlev, out.pos_row, out.level,
                                                                   out.depcnt, out.row_pos, cnt, ilev);
  DCHK(hipGetLastError());
  DCHK(rocprim::exclusive_scan(tmp, scan_bytes, cnt, out.off_ptr, 0, static_cast<size_t>(n) + 1,
                               rocprim::plus<int>(), s));
  // the level-ordered copy of the off-diagonal pattern
  k_offdiag<<<blocks(n), 256, 0, s>>>(n, unit_diag, row_ptr, col, out.pos_row, out.row_pos,
                                       out.off_ptr, out.off_col, out.off_pos, out.off_src,
                                       out.diag_src);
  DCHK(hipGetLastError());
  out.ilev.resize(static_cast<size_t>(nlev) + 1);
  int noff = 0;
  DCHK(hipMemcpyAsync(out.ilev.data(), ilev, (static_cast<size_t>(nlev) + 1) * sizeof(int),
                      hipMemcpyDeviceToHost, s));
  const bool near = max_len > kDefaultLaneEntries;
  if (near) {
    const int positions = (n + near_step(n) - 1) / near_step(n), per = 256 / kNearLanes;
    k_near<<<(positions + per - 1) / per, 256, 0, s>>>(n, near_step(n), out.pos_row, out.level,
                                                       out.off_ptr, out.off_col, tp.flags + 5);
    DCHK(hipGetLastError());
    DCHK(hipMemcpyAsync(got, tp.flags, sizeof(got), hipMemcpyDeviceToHost, s));
  } else {
    DCHK(hipMemcpyAsync(&noff, out.off_ptr + n, sizeof(int), hipMemcpyDeviceToHost, s));
  }
  DCHK(hipStreamSynchronize(s));
  if (near) {
    noff = got[7];
    out.near_row = static_cast<double>(got[5]) / ((n + near_step(n) - 1) / near_step(n));
    out.near_lane = static_cast<double>(got[5]) / got[6];
  }
  out.noff = noff;
  return kOk;
}

}  // namespace sptrsv

namespace sptrsv {

int device_transpose(int n, int64_t nnz, const int* row_ptr, const int* col, hipStream_t s,
                     int** rpT, int** colT, int** srcT) {
  *rpT = *colT = *srcT = nullptr;
  if (n < 1 || nnz < 0 || nnz > INT32_MAX) return kErrNotSupported;
  int *keys = nullptr, *keys_s = nullptr, *vals = nullptr, *row_of = nullptr;
  void* tmp = nullptr;
  int st = kOk;
  auto cleanup = [&]() {
    for (void* p : {static_cast<void*>(keys), static_cast<void*>(keys_s), static_cast<void*>(vals),
                    static_cast<void*>(row_of), tmp})
      dev_free(p);
  };
  if (dmalloc(&keys_s, nnz) || dmalloc(&vals, nnz) || dmalloc(&row_of, nnz) ||
      dmalloc(rpT, static_cast<int64_t>(n) + 1) || dmalloc(colT, nnz) || dmalloc(srcT, nnz)) {
    st = kErrOom;
  }
  int col_bits = 1;
  while (col_bits < 31 && (1ll << col_bits) < n) ++col_bits;
  if (!st && nnz > 0) {
    // entries by column, stably: (column, entry) ascending, i.e. the rows of
    // T^T with their columns (rows of T) strictly increasing
    if (dmalloc(&keys, nnz) ||
        hipMemcpyAsync(keys, col, static_cast<size_t>(nnz) * sizeof(int), hipMemcpyDeviceToDevice,
                       s) != hipSuccess) {
      st = kErrOom;
    } else {
      k_fill_iota<<<blocks(nnz), 256, 0, s>>>(vals, nnz);
      size_t tb = 0;
      if (rocprim::radix_sort_pairs(nullptr, tb, keys, keys_s, vals, *srcT,
                                    static_cast<unsigned>(nnz), 0, col_bits, s) != hipSuccess ||
          dev_alloc(&tmp, static_cast<int64_t>(tb)) != hipSuccess ||
          rocprim::radix_sort_pairs(tmp, tb, keys, keys_s, vals, *srcT, static_cast<unsigned>(nnz),
                                    0, col_bits, s) != hipSuccess)
        st = kErrHip;
    }
  }
  if (!st) {
    k_row_of<<<blocks(n), 256, 0, s>>>(n, row_ptr, row_of);
    k_transpose_fill<<<blocks(nnz > 0 ? nnz : 1), 256, 0, s>>>(n, nnz, keys_s, *srcT, row_of, *colT,
                                                               *rpT);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) st = kErrHip;
  }
  cleanup();
  if (st) {
    for (int** p : {rpT, colT, srcT})
      if (*p) {
        dev_free(*p);
        *p = nullptr;
      }
  }
  return st;
}

int device_value_sources(int n, int64_t noff_f, const int* off_src_f, const int* diag_src_f,
                         int64_t nnz, const int* srcT, DeviceAnalysis& t, hipStream_t s) {
  int* loc = nullptr;
  if (dmalloc(&loc, nnz)) return kErrOom;
  const int64_t tot_f = noff_f > n ? noff_f : n;
  const int64_t tot_t = t.noff > n ? t.noff : n;
  k_value_loc<<<blocks(tot_f), 256, 0, s>>>(n, noff_f, off_src_f, diag_src_f, loc);
  k_compose_src<<<blocks(tot_t), 256, 0, s>>>(n, t.noff, srcT, loc, t.off_src, t.diag_src);
  int st = kOk;
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) st = kErrHip;
  dev_free(loc);
  return st;
}

int device_concat(const std::vector<ConcatSystem>& systems, int vb, int* rp_cat, int* col_cat,
                  void* vals_cat, hipStream_t s) {
  const int count = static_cast<int>(systems.size());
  std::vector<SysDesc> host(count);
  int64_t roff = 0, eoff = 0, maxw = 1;
  for (int k = 0; k < count; ++k) {
    const ConcatSystem& c = systems[k];
    host[k] = SysDesc{c.row_ptr, c.col, c.vals, c.n, c.nnz, static_cast<int>(roff),
                      static_cast<int>(eoff)};
    roff += c.n;
    eoff += c.nnz;
    maxw = std::max<int64_t>(maxw, std::max<int64_t>(c.n, c.nnz));
  }
  SysDesc* dsys = nullptr;
  int* flags = nullptr;
  int st = kOk;
  if (dmalloc(&dsys, count) || dmalloc(&flags, 1)) st = kErrOom;
  int f = 0;
  if (!st && (hipMemcpyAsync(dsys, host.data(), count * sizeof(SysDesc), hipMemcpyHostToDevice, s) !=
                  hipSuccess ||
              hipMemsetAsync(flags, 0, sizeof(int), s) != hipSuccess))
    st = kErrHip;
  if (!st) {
    const int bx = static_cast<int>(std::min<int64_t>((maxw + 255) / 256, 1024));
    k_concat<<<dim3(bx, count), 256, 0, s>>>(dsys, vb, rp_cat, col_cat,
                                             static_cast<unsigned char*>(vals_cat), flags);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(&f, flags, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      st = kErrHip;
  }
  if (!st) {
    // the last row pointer: total nnz
    const int last = static_cast<int>(eoff);
    if (hipMemcpy(rp_cat + roff, &last, sizeof(int), hipMemcpyHostToDevice) != hipSuccess) st = kErrHip;
  }
  dev_free(dsys);
  dev_free(flags);
  if (!st && f) st = kErrNotSupported;
  return st;
}

}  // namespace sptrsv
