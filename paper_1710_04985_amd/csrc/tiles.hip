// Tiled self-scheduled solve: construction of the tiled copy, and the solve
// kernel (see tiles.hpp for the idea).
#include "tiles.hpp"

#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>

#include <algorithm>

#include "analysis.hpp"
#include "device_common.hpp"
#include "residency.hpp"

namespace sptrsv {
namespace {

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

// Adds d > 0 to an open-addressed table of kTileTable slots; false: no room.
__device__ __forceinline__ bool table_add(int* table, int d, bool agent) {
  unsigned h = (static_cast<unsigned>(d) * 2654435761u) >> 27;
  for (int probe = 0; probe < kTileTable; ++probe, h = (h + 1) & (kTileTable - 1)) {
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
// table, so that global atomics do not grow with the entries.
constexpr int kOffsetRows = 4096;

__global__ void __launch_bounds__(256)
k_tile_offsets(int n, const int* __restrict__ rp, const int* __restrict__ col, int nsys,
               const int* __restrict__ row0, int* table, int* full) {
  __shared__ int tab[kTileTable];
  __shared__ int over;
  const int r0 = blockIdx.x * kOffsetRows, r1 = min(n, r0 + kOffsetRows);
  int s = system_of(row0, nsys, r0);
  for (int a = r0; a < r1; ++s) {
    const int b = min(r1, row0[s + 1]);
    if (threadIdx.x < kTileTable) tab[threadIdx.x] = 0;
    if (threadIdx.x == 0) over = 0;
    __syncthreads();
    for (int i = a + threadIdx.x; i < b && !over; i += 256)
      for (int e = rp[i], e1 = rp[i + 1]; e < e1; ++e) {
        const int d = abs(col[e] - i);
        if (d != 0 && !table_add(tab, d, false)) {
          over = 1;
          break;
        }
      }
    __syncthreads();
    if (threadIdx.x < kTileTable) {
      const int d = tab[threadIdx.x];
      if (over || (d != 0 && !table_add(table + static_cast<int64_t>(s) * kTileTable, d, true)))
        __hip_atomic_store(full + s, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    a = b;
  }
}

__global__ void __launch_bounds__(256)
k_tile_lanes(int nchunks, const int* __restrict__ start, const int* __restrict__ meta,
             unsigned char* __restrict__ lanes_lg) {
  const int c = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, lane = threadIdx.x & 63;
  if (c >= nchunks) return;
  const int cnt = meta[c] & 0xffff, lg = meta[c] >> 16;
  for (int r = lane; r < cnt; r += 64) lanes_lg[start[c] + r] = static_cast<unsigned char>(lg);
}

// slot of entry e of a row with 2^lg partial sums (see k_tile)
__device__ __forceinline__ int entry_slot(int e, int lg, int acc) {
  return acc == 1 ? e : 4 * (e >> lg) + (e & ((1 << lg) - 1));
}

// counters of the construction
struct TileCount {
  int bad;      // an entry points ahead of its row's tile, or a table overflowed
  int ntiles;   // boxes that hold rows
  int slots;    // entry slots a row needs
  int last;     // largest sum of tile coordinates
};

// Every row: marks its box, and checks that each entry's tile is nowhere
// ahead of the row's own (so every entry leads to the same or an earlier tile
// of the order below).
__global__ void __launch_bounds__(256)
k_tile_mark(int n, const int* __restrict__ off_ptr, const int* __restrict__ off_col,
            const int* __restrict__ pos_row, const unsigned char* __restrict__ lanes_lg, int acc,
            const TileGrid* __restrict__ grids, int nsys, const int* __restrict__ row0,
            unsigned char* __restrict__ used, TileCount* cnt) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  int slots = 0;
  bool bad = false;
  if (k < n) {
    const int i = pos_row[k];
    const TileGrid& g = grids[nsys > 1 ? system_of(row0, nsys, i) : 0];
    const TilePoint p = tile_point(g, i - g.row0);
    const int t1 = p.c1 >> g.lx, t2 = p.c2 >> g.ly, t3 = p.c3 >> g.lz;
    const int box = tile_box(g, p);
    bad = box < 0 || box >= g.nbx * g.nby * g.nbz || tile_row(g, p) != i - g.row0;
    if (!bad) used[g.box0 + box] = 1;
    const int e0 = off_ptr[k], e1 = off_ptr[k + 1];
    for (int e = e0; e < e1; ++e) {
      const int j = off_col[e] - g.row0;
      if (j < 0 || j >= g.n) {
        bad = true;
        continue;
      }
      const TilePoint q = tile_point(g, j);
      bad |= (q.c1 >> g.lx) > t1 || (q.c2 >> g.ly) > t2 || (q.c3 >> g.lz) > t3;
    }
    const int lg = lanes_lg ? lanes_lg[k] : 0;
    if (e1 > e0) slots = entry_slot(e1 - e0 - 1, lg, acc) + 1;
    bad |= slots > kTileMaxEntries || lg > 2;
  }
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(&cnt->bad, 1);
  for (int o = 32; o > 0; o >>= 1) slots = max(slots, __shfl_xor(slots, o, 64));
  if ((threadIdx.x & 63) == 0 && slots > *const_cast<volatile int*>(&cnt->slots))
    atomicMax(&cnt->slots, slots);
}

// Order of the tiles: by the sum of their coordinates.  An entry's tile has
// no coordinate above its row's, so a different tile has a smaller sum.
__global__ void __launch_bounds__(256)
k_tile_keys(int nboxes, const TileGrid* __restrict__ grids, int nsys,
            const int* __restrict__ sys_box0, const unsigned char* __restrict__ used,
            unsigned* __restrict__ key, int* __restrict__ box_id, TileCount* cnt) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  bool u = false;
  if (b < nboxes) {
    const TileGrid& g = grids[nsys > 1 ? system_of(sys_box0, nsys, b) : 0];
    const TilePoint t = tile_of_box(g, b - g.box0);
    u = used[b] != 0;
    key[b] = u ? static_cast<unsigned>(t.c1 + t.c2 + t.c3) : 0x7fffffffu;
    box_id[b] = b;
  }
  const unsigned long long m = __ballot(u);
  if ((threadIdx.x & 63) == 0 && m) atomicAdd(&cnt->ntiles, __popcll(m));
  int last = u ? static_cast<int>(key[b]) : 0;
  for (int o = 32; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o, 64));
  if ((threadIdx.x & 63) == 0 && last) atomicMax(&cnt->last, last);
}

__global__ void __launch_bounds__(256)
k_tile_ranks(int ntiles, const int* __restrict__ sorted, int* __restrict__ box_tile) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < ntiles) box_tile[sorted[t]] = t;
}

// One wavefront per tile: the rows of its lanes, the LDS slot of every entry
// (a lane of the tile, a value from another tile, or the zero slot), the
// distinct external positions, and the number of levels inside the tile.
constexpr int kExtTable = 512;
constexpr int kZeroSlot = 255;
constexpr int kRowMask = (1 << 30) - 1;

__global__ void __launch_bounds__(64)
k_tile_build(const int* __restrict__ off_ptr, const int* __restrict__ off_col,
             const int* __restrict__ row_pos, const unsigned char* __restrict__ lanes_lg, int acc,
             const TileGrid* __restrict__ grids, int nsys, const int* __restrict__ sys_box0,
             const int* __restrict__ sorted, const int* __restrict__ box_tile, int E, int X,
             DevTiles d, TileCount* cnt) {
  __shared__ int htab[kExtTable];      // external position + 1, 0 = empty
  __shared__ int hidx[kExtTable];      // its place in the tile's list
  __shared__ int lev[64];
  const int t = blockIdx.x, lane = threadIdx.x;
  for (int h = lane; h < kExtTable; h += 64) htab[h] = 0;
  __syncthreads();
  const int box = sorted[t];
  const TileGrid& g = grids[nsys > 1 ? system_of(sys_box0, nsys, box) : 0];
  const TilePoint tp = tile_of_box(g, box - g.box0);
  const int r = tile_row(g, tile_lane_point(g, tp, lane));
  const int k = r >= 0 ? row_pos[g.row0 + r] : -1;
  const int e0 = k >= 0 ? off_ptr[k] : 0, len = k >= 0 ? off_ptr[k + 1] - e0 : 0;
  const int lg = k >= 0 && lanes_lg ? lanes_lg[k] : 0;
  // byte per entry slot: lane of the tile, 64 + table slot (resolved below),
  // kZeroSlot
  int where[kTileMaxEntries];          // table slot of an external value, -1 - lane inside
  bool bad = false;
#pragma unroll
  for (int e = 0; e < kTileMaxEntries; ++e) {
    where[e] = INT32_MIN;
    if (e >= len) continue;
    const TilePoint q = tile_point(g, off_col[e0 + e] - g.row0);
    const int qb = g.box0 + tile_box(g, q), ql = tile_lane(g, q);
    if (qb == box) {
      where[e] = -1 - ql;
      continue;
    }
    const int pos = box_tile[qb] * 64 + ql;
    // the table is addressed by the low bits of the position, so the list
    // comes out nearly in position order and neighbouring lanes poll
    // neighbouring values
    int h = pos & (kExtTable - 1), probe = 0;
    for (; probe < kExtTable; ++probe, h = (h + 1) & (kExtTable - 1)) {
      const int v = atomicCAS(htab + h, 0, pos + 1);
      if (v == 0 || v == pos + 1) break;
    }
    if (probe == kExtTable) bad = true;
    where[e] = h;
  }
  __syncthreads();
  // places in the list: occupied slots in table order
  int mine = 0;
#pragma unroll
  for (int u = 0; u < kExtTable / 64; ++u) mine += htab[lane * (kExtTable / 64) + u] != 0;
  int incl = mine;
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  const int total = __shfl(incl, 63, 64);
  if (total > kTileMaxExt || total > 64 * X) bad = true;
  for (int w = lane; w < 64 * X; w += 64) d.epos[static_cast<int64_t>(t) * X * 64 + w] = -1;
  __syncthreads();
  int at = incl - mine;
#pragma unroll
  for (int u = 0; u < kExtTable / 64; ++u) {
    const int h = lane * (kExtTable / 64) + u, v = htab[h];
    hidx[h] = at;
    if (v != 0) {
      if (at < 64 * X) d.epos[static_cast<int64_t>(t) * X * 64 + at] = v - 1;
      ++at;
    }
  }
  __syncthreads();
  // slots and value sources
  for (int q = 0; q < E; ++q) d.src[(static_cast<int64_t>(t) * E + q) * 64 + lane] = -1;
  unsigned words[(kTileMaxEntries + 3) / 4];
#pragma unroll
  for (int w = 0; w < (kTileMaxEntries + 3) / 4; ++w) words[w] = 0xffffffffu;
#pragma unroll
  for (int e = 0; e < kTileMaxEntries; ++e) {
    if (e >= len) continue;
    const int q = entry_slot(e, lg, acc);
    const int sl = where[e] < 0 ? -1 - where[e] : 64 + hidx[where[e]];
    if (q >= E || sl >= kZeroSlot) {
      bad = true;
      continue;
    }
#pragma unroll
    for (int w = 0; w < (kTileMaxEntries + 3) / 4; ++w)
      if (w == (q >> 2))
        words[w] = (words[w] & ~(0xffu << (8 * (q & 3)))) | (static_cast<unsigned>(sl) << (8 * (q & 3)));
    d.src[(static_cast<int64_t>(t) * E + q) * 64 + lane] = e0 + e;
  }
  const int NW = (E + 3) / 4;
#pragma unroll
  for (int w = 0; w < (kTileMaxEntries + 3) / 4; ++w)
    if (w < NW) d.slot[(static_cast<int64_t>(t) * NW + w) * 64 + lane] = words[w];
  // the row, with the row's log2 of partial sums in the top two bits
  d.row[static_cast<int64_t>(t) * 64 + lane] =
      r >= 0 ? static_cast<int>(static_cast<unsigned>(g.row0 + r) | (static_cast<unsigned>(lg) << 30))
             : -1;
  d.dsrc[static_cast<int64_t>(t) * 64 + lane] = k;
  // levels inside the tile
  int my = 1;
  for (;;) {
    lev[lane] = my;
    __syncthreads();
    int up = 1;
#pragma unroll
    for (int e = 0; e < kTileMaxEntries; ++e)
      if (e < len && where[e] < 0) up = max(up, 1 + lev[-1 - where[e]]);
    up = min(up, 64);
    const bool again = __any(up != my);
    __syncthreads();
    if (!again) break;
    my = up;
  }
  for (int o = 32; o > 0; o >>= 1) my = max(my, __shfl_xor(my, o, 64));
  if (lane == 0) d.depth[t] = my;
  if (__any(bad) && lane == 0) atomicOr(&cnt->bad, 1);
}

// values of the tiled copy: entries it lacks are -0, whose product with the
// zero slot (+0) is -0 and changes no sum
template <typename T>
__global__ void __launch_bounds__(256)
k_tile_gather(int64_t nval, int64_t npos, const int* __restrict__ src, const int* __restrict__ dsrc,
              const T* __restrict__ off_val, const T* __restrict__ dinv, T* __restrict__ tval,
              T* __restrict__ tdinv) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; q < nval + npos;
       q += stride) {
    if (q < nval) {
      const int s = src[q];
      tval[q] = s >= 0 ? off_val[s] : -T(0);
    } else {
      const int s = dsrc[q - nval];
      tdinv[q - nval] = s >= 0 ? dinv[s] : T(1);
    }
  }
}

// -------------------------------------------------------------------- solve

template <typename T> struct TArgs {
  int ntiles;
  const int* row;
  const int* depth;
  const unsigned* slot;
  const int* epos;
  const T* val;
  const T* dinv;
  const T* b;
  T* x;
  T* xp;
  int* status;
  int* arrive;
  int spin_limit;
  int res_limit;
};

// Bounded wait for the values at e[0..X) of xp (-1: none).  Two rounds
// overlap, as in the row-wise kernels: the second is issued before the first
// is looked at, so a value is seen about half a round trip after it lands.
// After spin_limit rounds, or once another wavefront has timed out, TIMEOUT is
// raised and the missing values become quiet NaNs, so the grid drains.
template <typename T, int X>
__device__ __forceinline__ void wait_ext(const T* xp, const int (&e)[X], T (&v)[X], int spin_limit,
                                         int* status) {
  const T* p[X];
  unsigned pend = 0;
#pragma unroll
  for (int q = 0; q < X; ++q) {
    p[q] = xp + (e[q] >= 0 ? e[q] : 0);
    v[q] = T(0);
    if (e[q] >= 0) pend |= 1u << q;
  }
  auto take = [&](const T (&w)[X]) {
#pragma unroll
    for (int q = 0; q < X; ++q)
      if (((pend >> q) & 1u) && !is_sentinel(w[q])) {
        v[q] = w[q];
        pend &= ~(1u << q);
      }
  };
  if (!pend) return;
  T pa[X], pb[X];
#pragma unroll
  for (int q = 0; q < X; ++q) pa[q] = load_agent(p[q]);
  for (int s = 1; s <= spin_limit; s += 2) {
    __builtin_amdgcn_s_sleep(1);
#pragma unroll
    for (int q = 0; q < X; ++q) pb[q] = load_agent(p[q]);
    take(pa);
    if (!pend) return;
    __builtin_amdgcn_s_sleep(1);
#pragma unroll
    for (int q = 0; q < X; ++q) pa[q] = load_agent(p[q]);
    take(pb);
    if (!pend) return;
    if ((s & 63) == 63 && (load_status(status) & kStatusTimeout)) break;
  }
  raise_status(status, kStatusTimeout);
#pragma unroll
  for (int q = 0; q < X; ++q)
    if ((pend >> q) & 1u) v[q] = __builtin_nan("");
}

// Bound by the chain of tiles: one hop (about 0.6 us with its polls) plus the
// tile's own levels (about 70 ns each: LDS reads, FMAs, LDS write) per tile of
// the chain; 128^3 7-point, lower then upper: 340 us a step against 772 with
// a hop per level, 1024^2 9-point 1271 against 5032, 128^3 27-point 970
// against 4402, 256 2-D ILU(0) factors 198 against 582.
//
// Tile t goes to wavefront t mod W of an all-resident grid.  Tiles are in
// dependency order, so the wavefront of the lowest unfinished tile is working
// on it and the tile's dependencies are done: the grid always progresses.
//
// Inside a tile every lane recomputes its row once per level of the tile from
// the LDS copy of x: after s rounds the rows of the first s levels hold their
// final value, and recomputing a final row gives the same bits, so no lane
// needs to know its level.  Entries are summed in stored order with FMA; with
// A = 4 slot q adds to partial sum q mod 4, which are then added in the
// order of the row-wise kernels' butterfly (rows that those kernels give
// fewer lanes leave the upper sums at -0, which changes nothing): the same
// bits as every other schedule.
template <typename T, int E, int X, int A>
__global__ void __launch_bounds__(64) k_tile(TArgs<T> a) {
  __shared__ T xs[256];
  constexpr int NW = (E + 3) / 4;
  const int lane = threadIdx.x;
  if (!grid_resident(a.arrive, a.res_limit, a.status)) return;
  const int W = gridDim.x;
  if (lane == 0) xs[kZeroSlot] = T(0);
  struct Stage {
    int row, depth;
    int e[X];
    unsigned w[NW];
    T v[E], d, b;
  };
  // loads of tile t (clamped past the end; its b needs the row number, loaded
  // one tile earlier)
  auto load = [&](Stage& s, int t, int row) {
    const int64_t tc = t < a.ntiles ? t : a.ntiles - 1;
    s.row = row;
    s.depth = a.depth[tc];
#pragma unroll
    for (int q = 0; q < X; ++q) s.e[q] = a.epos[(tc * X + q) * 64 + lane];
#pragma unroll
    for (int q = 0; q < NW; ++q) s.w[q] = a.slot[(tc * NW + q) * 64 + lane];
#pragma unroll
    for (int q = 0; q < E; ++q) s.v[q] = a.val[(tc * E + q) * 64 + lane];
    s.d = a.dinv[tc * 64 + lane];
    s.b = a.b[row != -1 ? row & kRowMask : 0];
  };
  auto row_of = [&](int t) {
    const int64_t tc = t < a.ntiles ? t : a.ntiles - 1;
    return a.row[tc * 64 + lane];
  };
  Stage cur;
  load(cur, blockIdx.x, row_of(blockIdx.x));
  int row_next = row_of(blockIdx.x + W);
  for (int t = blockIdx.x; t < a.ntiles; t += W) {
    T ev[X];
    wait_ext<T, X>(a.xp, cur.e, ev, a.spin_limit, a.status);
    Stage nxt;
    load(nxt, t + W, row_next);
    row_next = row_of(t + 2 * W < t ? a.ntiles : t + 2 * W);
#pragma unroll
    for (int q = 0; q < X; ++q) xs[64 + 64 * q + lane] = ev[q];
    int at[E];
#pragma unroll
    for (int q = 0; q < E; ++q) at[q] = (cur.w[q >> 2] >> (8 * (q & 3))) & 0xff;
    T init[A];
#pragma unroll
    for (int q = 0; q < A; ++q) init[q] = q < (1 << (cur.row >> 30 & 3)) ? T(0) : -T(0);
    const int depth = wave_uniform(cur.depth);
    T xi = T(0);
    for (int s = 0; s < depth; ++s) {
      // one wavefront's LDS accesses are performed in issue order; the fence
      // keeps the compiler from moving them (it emits nothing)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      T g[E];
#pragma unroll
      for (int q = 0; q < E; ++q) g[q] = xs[at[q]];
      T sum[A];
#pragma unroll
      for (int q = 0; q < A; ++q) sum[q] = init[q];
#pragma unroll
      for (int q = 0; q < E; ++q) sum[q % A] = fma_t(cur.v[q], g[q], sum[q % A]);
      T tot = sum[0];
      if constexpr (A == 4) tot = (sum[0] + sum[1]) + (sum[2] + sum[3]);
      xi = canonical((cur.b - tot) * cur.d);
      xs[lane] = xi;
    }
    store_agent(a.xp + static_cast<int64_t>(t) * 64 + lane, xi);
    if (cur.row != -1) a.x[cur.row & kRowMask] = xi;
    cur = nxt;
  }
}

template <typename T> const void* tile_fn(const DevTiles& t) {
#define SPTRSV_TILE(E, X, A)                               \
  if (t.entries == E && t.ext == X && t.acc == A)          \
  return reinterpret_cast<const void*>(k_tile<T, E, X, A>)
  SPTRSV_TILE(2, 1, 1);
  SPTRSV_TILE(3, 1, 1);
  SPTRSV_TILE(4, 1, 1);
  SPTRSV_TILE(2, 2, 1);
  SPTRSV_TILE(3, 2, 1);
  SPTRSV_TILE(4, 2, 1);
  SPTRSV_TILE(2, 3, 1);
  SPTRSV_TILE(3, 3, 1);
  SPTRSV_TILE(4, 3, 1);
  SPTRSV_TILE(13, 1, 4);
  SPTRSV_TILE(13, 2, 4);
  SPTRSV_TILE(13, 3, 4);
  SPTRSV_TILE(16, 1, 4);
  SPTRSV_TILE(16, 2, 4);
  SPTRSV_TILE(16, 3, 4);
#undef SPTRSV_TILE
  return nullptr;
}

inline int blocks(int64_t work, int per) {
  const int64_t b = (work + per - 1) / per;
  return static_cast<int>(b < 1 ? 1 : b < (1 << 30) ? b : (1 << 30));
}

struct DevFree {
  std::vector<void*> p;
  ~DevFree() {
    for (void* q : p)
      if (q) (void)hipFree(q);
  }
  template <typename T> bool get(T** out, int64_t count) {
    void* q = nullptr;
    if (hipMalloc(&q, static_cast<size_t>(count > 0 ? count : 1) * sizeof(T)) != hipSuccess)
      return false;
    p.push_back(q);
    *out = static_cast<T*>(q);
    return true;
  }
};

}  // namespace

hipError_t launch_tile_offsets(int n, const int* row_ptr, const int* col, int nsys,
                               const int* sys_row0, int* table, int* full, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_tile_offsets<<<blocks(n, kOffsetRows), 256, 0, s>>>(n, row_ptr, col, nsys, sys_row0, table,
                                                        full);
  return hipGetLastError();
}

hipError_t launch_tile_lanes(const DevChunks& c, unsigned char* lanes_lg, hipStream_t s) {
  if (c.count == 0) return hipSuccess;
  k_tile_lanes<<<blocks(static_cast<int64_t>(c.count) * 64, 256), 256, 0, s>>>(c.count, c.start,
                                                                              c.meta, lanes_lg);
  return hipGetLastError();
}

template <typename T> hipError_t launch_tile_gather(const DevPlan& p, const DevTiles& t,
                                                    hipStream_t s) {
  const int64_t nval = t.npos * t.entries;
  if (t.npos == 0) return hipSuccess;
  k_tile_gather<T><<<blocks(nval + t.npos, 256), 256, 0, s>>>(
      nval, t.npos, t.src, t.dsrc, static_cast<const T*>(p.off_val), static_cast<const T*>(p.dinv),
      static_cast<T*>(t.val), static_cast<T*>(t.dinv));
  return hipGetLastError();
}

void free_tiles(DevTiles& t) {
  if (t.mem) (void)hipFree(t.mem);
  t = DevTiles();
}

int build_tiles(const DevPlan& p, const std::vector<TileGrid>& grids, int ext, int max_len,
                const unsigned char* lanes_lg, int vb, hipStream_t s, DevTiles& out) {
  out = DevTiles();
  const int nsys = static_cast<int>(grids.size());
  if (p.n == 0 || nsys == 0 || ext > kTileMaxExt || max_len > kTileMaxEntries || !p.row_pos)
    return kErrNotSupported;
  int64_t nboxes = 0;
  std::vector<int> row0(nsys + 1), box0(nsys + 1);
  std::vector<TileGrid> gh(grids);
  for (int k = 0; k < nsys; ++k) {
    gh[k].box0 = static_cast<int>(nboxes);
    row0[k] = gh[k].row0;
    box0[k] = gh[k].box0;
    nboxes += gh[k].n > 0 ? static_cast<int64_t>(gh[k].nbx) * gh[k].nby * gh[k].nbz : 0;
    if (nboxes > (1 << 24)) return kErrNotSupported;   // positions stay well inside 32 bits
  }
  row0[nsys] = p.n;
  box0[nsys] = static_cast<int>(nboxes);
  const int acc = lanes_lg ? 4 : 1;
  DevFree f;
  TileGrid* grids_d = nullptr;
  int *row0_d = nullptr, *box0_d = nullptr, *box_id = nullptr, *sorted = nullptr, *box_tile = nullptr;
  unsigned char* used = nullptr;
  unsigned *key = nullptr, *key_s = nullptr;
  TileCount* cnt = nullptr;
  if (!f.get(&grids_d, nsys) || !f.get(&row0_d, nsys + 1) || !f.get(&box0_d, nsys + 1) ||
      !f.get(&box_id, nboxes) || !f.get(&sorted, nboxes) || !f.get(&box_tile, nboxes) ||
      !f.get(&used, nboxes) || !f.get(&key, nboxes) || !f.get(&key_s, nboxes) || !f.get(&cnt, 1))
    return kErrOom;
  TileCount c{0, 0, 0, 0};
#define TCHK(expr)                                \
  do {                                            \
    if ((expr) != hipSuccess) return kErrHip;     \
  } while (0)
  TCHK(hipMemcpyAsync(grids_d, gh.data(), nsys * sizeof(TileGrid), hipMemcpyHostToDevice, s));
  TCHK(hipMemcpyAsync(row0_d, row0.data(), (nsys + 1) * sizeof(int), hipMemcpyHostToDevice, s));
  TCHK(hipMemcpyAsync(box0_d, box0.data(), (nsys + 1) * sizeof(int), hipMemcpyHostToDevice, s));
  TCHK(hipMemcpyAsync(cnt, &c, sizeof(c), hipMemcpyHostToDevice, s));
  TCHK(hipMemsetAsync(used, 0, static_cast<size_t>(nboxes), s));
  k_tile_mark<<<blocks(p.n, 256), 256, 0, s>>>(p.n, p.off_ptr, p.off_col, p.pos_row, lanes_lg, acc,
                                              grids_d, nsys, row0_d, used, cnt);
  TCHK(hipGetLastError());
  k_tile_keys<<<blocks(nboxes, 256), 256, 0, s>>>(static_cast<int>(nboxes), grids_d, nsys, box0_d,
                                                 used, key, box_id, cnt);
  TCHK(hipGetLastError());
  size_t tb = 0;
  TCHK(rocprim::radix_sort_pairs(nullptr, tb, key, key_s, box_id, sorted,
                                 static_cast<unsigned>(nboxes), 0, 31, s));
  unsigned char* tmp = nullptr;
  if (!f.get(&tmp, static_cast<int64_t>(tb))) return kErrOom;
  TCHK(rocprim::radix_sort_pairs(tmp, tb, key, key_s, box_id, sorted,
                                 static_cast<unsigned>(nboxes), 0, 31, s));
  TCHK(hipMemcpyAsync(&c, cnt, sizeof(c), hipMemcpyDeviceToHost, s));
  TCHK(hipStreamSynchronize(s));
  if (c.bad || c.ntiles < 1) return kErrNotSupported;
  DevTiles t;
  t.ntiles = c.ntiles;
  t.order = c.last + 1;
  t.npos = static_cast<int64_t>(c.ntiles) * 64;
  t.acc = acc;
  t.entries = acc == 1 ? std::max(2, c.slots) : c.slots <= 13 ? 13 : 16;
  t.ext = std::max(1, (ext + 63) / 64);
  if (t.entries > (acc == 1 ? 4 : 16)) return kErrNotSupported;
  const int E = t.entries, X = t.ext, NW = (E + 3) / 4;
  const int64_t np = t.npos;
  // one allocation: values first (8-byte aligned), then the index arrays
  const int64_t bytes = np * (E + 1) * vb + np * 4 * (1 + NW + X + E + 1) + t.ntiles * 4ll;
  if (hipMalloc(&t.mem, static_cast<size_t>(bytes)) != hipSuccess) return kErrOom;
  char* at = static_cast<char*>(t.mem);
  auto take = [&](int64_t b) {
    char* q = at;
    at += b;
    return q;
  };
  t.val = take(np * E * vb);
  t.dinv = take(np * vb);
  t.row = reinterpret_cast<int*>(take(np * 4));
  t.slot = reinterpret_cast<unsigned*>(take(np * 4 * NW));
  t.epos = reinterpret_cast<int*>(take(np * 4 * X));
  t.src = reinterpret_cast<int*>(take(np * 4 * E));
  t.dsrc = reinterpret_cast<int*>(take(np * 4));
  t.depth = reinterpret_cast<int*>(take(t.ntiles * 4ll));
  k_tile_ranks<<<blocks(t.ntiles, 256), 256, 0, s>>>(t.ntiles, sorted, box_tile);
  k_tile_build<<<t.ntiles, 64, 0, s>>>(p.off_ptr, p.off_col, p.row_pos, lanes_lg, acc, grids_d,
                                       nsys, box0_d, sorted, box_tile, E, X, t, cnt);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(&c, cnt, sizeof(c), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess || c.bad) {
    free_tiles(t);
    return e != hipSuccess ? kErrHip : kErrNotSupported;
  }
#undef TCHK
  out = t;
  return kOk;
}

template <typename T> hipError_t launch_tile_solve(const TileSolveArgs& sa, hipStream_t s) {
  const DevTiles& t = *sa.tiles;
  if (t.ntiles == 0) return hipSuccess;
  TArgs<T> a;
  a.ntiles = t.ntiles;
  a.row = t.row;
  a.depth = t.depth;
  a.slot = t.slot;
  a.epos = t.epos;
  a.val = static_cast<const T*>(t.val);
  a.dinv = static_cast<const T*>(t.dinv);
  a.b = static_cast<const T*>(sa.b);
  a.x = static_cast<T*>(sa.x);
  a.xp = static_cast<T*>(sa.xp);
  a.status = sa.scratch.status;
  a.arrive = sa.scratch.arrive;
  a.spin_limit = sa.spin_limit;
  a.res_limit = sa.res_limit;
  const void* fn = tile_fn<T>(t);
  if (!fn) return hipErrorInvalidValue;
  void* args[] = {&a};
  if (sa.coop) return hipLaunchCooperativeKernel(fn, dim3(sa.grid), dim3(64), args, 0, s);
  return hipLaunchKernel(fn, dim3(sa.grid), dim3(64), args, 0, s);
}

template <typename T> int tile_blocks_per_cu(const DevTiles& t) {
  const void* fn = tile_fn<T>(t);
  int nb = 0;
  if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, 64, 0) != hipSuccess) return 1;
  return nb > 0 ? nb : 1;
}

#define SPTRSV_INSTANTIATE(T)                                                                  \
  template hipError_t launch_tile_gather<T>(const DevPlan&, const DevTiles&, hipStream_t);     \
  template hipError_t launch_tile_solve<T>(const TileSolveArgs&, hipStream_t);                 \
  template int tile_blocks_per_cu<T>(const DevTiles&);

SPTRSV_INSTANTIATE(double)
SPTRSV_INSTANTIATE(float)

}  // namespace sptrsv
