// The filter stage of Section 4.1 on the device: candidate pairs of two
// polygon sets are the pairs whose MBRs intersect.  Per set, a uniform grid
// over the extent of the set's A polygons indexes them (a counting sort of
// (cell, polygon) entries); each B polygon visits the cells its MBR covers
// and keeps the A polygons whose MBR shares a pixel with its own, reporting
// a pair only from the cell that holds the lower-left pixel of the two MBRs'
// intersection, so that every pair is found once.  Each B polygon's pairs are
// written to a segment of their own (offsets from a scan of the counts) in
// the order of A: the output is ordered by set, then B, then A.
//
// All of it is queued without a look at the sizes it finds on the way (cells,
// entries, pairs): the kernels take them from device memory and stop where
// one exceeds the room for it, and the host reads them once, at the end.
#include <limits.h>

#include <algorithm>

#include "sccg_device.h"

namespace sccg {

namespace {

// The set holding index k: the largest s with off[s] <= k, or -1 when k lies
// outside [off[0], off[n]).
__device__ __forceinline__ int64_t set_of(const int64_t* off, int64_t n, int64_t k) {
  if (n <= 0 || k < off[0] || k >= off[n]) return -1;
  int64_t lo = 0, hi = n;  // off[lo] <= k < off[hi]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (off[mid] <= k)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The same from set lo on: off[lo] <= k < off[n].
__device__ __forceinline__ int64_t set_from(const int64_t* off, int64_t n, int64_t lo, int64_t k) {
  int64_t step = 1;
  while (lo + step < n && off[lo + step] <= k) {
    lo += step;
    step *= 2;
  }
  int64_t hi = min(lo + step, n);
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (off[mid] <= k)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The same for every lane's k, ascending over the wave (a lane without one
// passes -1): the set of the first is searched by the wave, 64 offsets per
// step, the others from it in steps that double (most are in the same set or
// the next; a walk over the sets between took 89 ms for 100 polygons in a
// million sets).  Every lane takes part.
__device__ __forceinline__ int64_t set_of_lane(const int64_t* off, int64_t n, int64_t k) {
  const int lane = lane_id();
  const uint64_t some = ballot(n > 0 && k >= off[0] && k < off[n]);
  if (!some) return -1;
  const int64_t k0 = uniform64(__shfl((long long)k, __ffsll((long long)some) - 1, kWave));
  int64_t lo = 0, hi = n;  // off[lo] <= k0 < off[hi]
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + kWave - 1) / kWave;
    const uint64_t m = ballot(lo + lane * step < hi && off[min(lo + lane * step, hi - 1)] <= k0);
    lo = uniform64(lo + (__popcll(m) - 1) * step);
    hi = uniform64(min(hi, lo + step));
  }
  if (!((some >> lane) & 1ull)) return -1;
  return set_from(off, n, lo, k);
}

__device__ __forceinline__ bool meta_empty(const Meta& m) { return m.x0 >= m.x1 || m.y0 >= m.y1; }

// cell index of pixel coordinate v in a grid starting at o (floor division,
// v >= o); v - o can reach 2^31 with coordinates up to 2^30 in size
__device__ __forceinline__ int cell_of(int v, int o, int cell) {
  return (int)(((uint32_t)v - (uint32_t)o) / (uint32_t)cell);
}

}  // namespace

__device__ __forceinline__ int4 no_extent() { return make_int4(INT_MAX, INT_MAX, INT_MIN, INT_MIN); }
__global__ void k_join_init_sets(int64_t n_sets, int4* bbox) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n_sets) bbox[s] = no_extent();
}

// Extent of each set's A polygons.  Sets are contiguous ranges: a workgroup
// takes kBoxRun consecutive polygons, a thread up to 16 neighbouring ones
// of them (through LDS), and a set is updated by a thread when it leaves it and by the
// workgroup for the threads that end in the same one.  (The atomics on one
// set's extent take turns: 600,000 polygons of 16 sets took 250 us with four
// for every 64 polygons, 55 for every 256, 23 for every 1024.  A workgroup that
// took one set after the other needed 1.4 us for each: 370 us, now 9, for 4096
// polygons of 256 sets.)
constexpr int kBoxRun = 4096;
// What the waves' last sets come to: one per wave, -1 where its threads differ.
struct WaveBox {
  int64_t set;
  int4 box;
};
__device__ __forceinline__ int4 box_or(const int4& a, const int4& b) {
  return make_int4(min(a.x, b.x), min(a.y, b.y), max(a.z, b.z), max(a.w, b.w));
}
// add(s, box): the polygons [a0, a1), a1 - a0 <= kBoxRun, of set s (by any
// thread, several times a set).
// Whether the lanes' sets (ascending, -1 for none) are one; then every lane has
// it and the extent of all.  Else the first lane of each set has its lanes', the
// others nothing (one by one the atomics of 16 such waves took 18 us).
__device__ __forceinline__ bool one_set(int64_t& s, int4& box) {
  const uint64_t some = ballot(s >= 0);
  if (s < 0) box = no_extent();
  const int64_t s0 = some ? uniform64(__shfl((long long)s, __ffsll((long long)some) - 1, kWave)) : -1;
  if (ballot(s >= 0 && s != s0) == 0) {
    s = s0;
    box = make_int4(wave_min_i32(box.x), wave_min_i32(box.y), wave_max_i32(box.z), wave_max_i32(box.w));
    return true;
  }
  const int lane = lane_id(), mine = (int)s;
  for (int d = 1; d < kWave; d <<= 1) {
    const int4 o = make_int4(__shfl_down(box.x, d, kWave), __shfl_down(box.y, d, kWave), __shfl_down(box.z, d, kWave),
                             __shfl_down(box.w, d, kWave));
    const bool same = __shfl_down(mine, d, kWave) == mine;
    if (same && lane + d < kWave) box = box_or(box, o);
  }
  const int before = __shfl_up(mine, 1, kWave);
  if (lane > 0 && before == mine) s = -1;
  return false;
}
template <int kThreads, int kRun>
struct RunLds {
  int4 meta[kRun + kThreads];  // an entry between two threads' polygons: their banks differ
  WaveBox wave[kThreads / kWave];
};
template <int kThreads, int kRun, typename F>
__device__ __forceinline__ void run_extents(int64_t a0, int64_t a1, const Meta* metaA, const int64_t* a_off,
                                            int64_t n_sets, RunLds<kThreads, kRun>& lds, F add) {
  const int t = (int)threadIdx.x, w = t / kWave;
  const int cnt = (int)(a1 - a0);
  int sh = 0;  // 2^sh polygons a thread
  while ((kThreads << sh) < cnt) ++sh;
#pragma unroll 4
  for (int i = t; i < cnt; i += kThreads) {
    const Meta m = load_meta(metaA, a0 + i);
    lds.meta[i + (i >> sh)] = make_int4(m.x0, m.y0, m.x1, m.y1);
  }
  // the thread's polygons [a, end) that are in a set
  const int64_t first = n_sets > 0 ? a_off[0] : a1, last = n_sets > 0 ? a_off[n_sets] : a0;
  const int64_t b = a0 + (t << sh), a = max(b, first), end = min(min(b + (1 << sh), a1), last);
  int64_t s = set_of_lane(a_off, n_sets, a < end ? a : -1), s_end = s >= 0 ? a_off[s + 1] : 0;
  int4 box = no_extent();
  __syncthreads();
#pragma unroll 1
  for (int64_t k = a; k < end; ++k) {
    if (k >= s_end) {
      if (box.x < box.z) add(s, box);
      box = no_extent();
      s = set_from(a_off, n_sets, s, k);
      s_end = a_off[s + 1];
    }
    const int4 m = lds.meta[(t << sh) + t + (int)(k - b)];
    if (m.x < m.z && m.y < m.w) box = box_or(box, m);
  }
  // the threads' last sets: a wave that has one only leaves it to the workgroup
  if (one_set(s, box)) {
    if (lane_id() == 0) lds.wave[w] = WaveBox{s, box};
  } else {
    if (s >= 0 && box.x < box.z) add(s, box);
    if (lane_id() == 0) lds.wave[w] = WaveBox{-1, box};
  }
  __syncthreads();
  if (w == 0) {
    const int l = min(lane_id(), kThreads / kWave - 1);
    s = lds.wave[l].set;
    box = lds.wave[l].box;
    if (lane_id() != l) s = -1;
    if (one_set(s, box)) s = lane_id() == 0 ? s : -1;
    if (s >= 0 && box.x < box.z) add(s, box);
  }
}
__device__ __forceinline__ void add_extent(int4* to, const int4& m) {
  atomicMin(&to->x, m.x);
  atomicMin(&to->y, m.y);
  atomicMax(&to->z, m.z);
  atomicMax(&to->w, m.w);
}
template <int kRun>
__global__ void __launch_bounds__(256) k_join_bbox(Polys A, const Meta* metaA, const int64_t* a_off, int64_t n_sets,
                                                   int4* bbox) {
  __shared__ RunLds<256, kRun> lds;
  const int64_t a0 = (int64_t)blockIdx.x * kRun;
  run_extents<256, kRun>(a0, min(a0 + kRun, A.n), metaA, a_off, n_sets, lds,
                         [&](int64_t s, const int4& m) { add_extent(bbox + s, m); });
}
// Of sets of fewer polygons on average a thread takes one polygon, not several
// sets (runs of 4096 / 256 polygons, 600,000 of them in sets of 600: 8.0 / 9.4 us;
// of 100: 14 / 11; of 10: 17.5 / 12; a million in sets of one: 157 / 49).
constexpr int64_t kSmallSets = 128;
constexpr int kSmallRun = 256;

// ------------------------------------------------------- exclusive scans
// exclusive prefix of v over the threads of a block (kThreads of them; sh: one per wave)
constexpr int kScanThreads = 256;
constexpr int kScanPer = 8;
constexpr int kScanBlock = kScanThreads * kScanPer;
template <int kThreads = kScanThreads>
__device__ __forceinline__ int64_t block_exclusive(int64_t v, int64_t* sh, int64_t* total) {
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  int64_t x = v;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int64_t u = __shfl_up((long long)x, d, kWave);
    if (lane >= d) x += u;
  }
  if (lane == kWave - 1) sh[w] = x;
  __syncthreads();
  int64_t before = 0, all = 0;
  for (int k = 0; k < kThreads / kWave; ++k) {
    before += k < w ? sh[k] : 0;
    all += sh[k];
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// Grid of set s: origin, columns, rows.  Returns its cells.
__device__ __forceinline__ int64_t set_grid(int64_t s, const int4* bbox, int cell, int4* grid, uint32_t* err) {
  const int4 b = bbox[s];
  int gw = 0, gh = 0;
  if (b.x < b.z && b.y < b.w) {
    const int64_t w = ((int64_t)b.z - b.x + cell - 1) / cell, h = ((int64_t)b.w - b.y + cell - 1) / cell;
    if (w * h > (1 << 24)) {
      latch_error(err, kErrSide);  // the set's grid is too large for the cell size
    } else {
      gw = (int)w;
      gh = (int)h;
    }
  }
  grid[s] = make_int4(b.x, b.y, gw, gh);
  return (int64_t)gw * gh;
}
// The grids of all sets by one block; base[s] = cells of the sets before s,
// base[n_sets] = all of them.
template <int kThreads>
__device__ __forceinline__ void set_grids(int64_t n_sets, const int4* bbox, int cell, int4* grid, int64_t* base,
                                          uint32_t* err, int64_t* sh) {
  int64_t run = 0;
  for (int64_t s0 = 0; s0 < n_sets; s0 += kThreads) {
    const int64_t s = s0 + threadIdx.x;
    const int64_t cells = s < n_sets ? set_grid(s, bbox, cell, grid, err) : 0;
    int64_t total;
    const int64_t before = block_exclusive<kThreads>(cells, sh, &total);
    if (s < n_sets) base[s] = run + before;
    run += total;
  }
  if (threadIdx.x == 0) base[n_sets] = run;
}
__global__ void __launch_bounds__(kScanThreads) k_join_grid(int64_t n_sets, const int4* bbox, int cell, int4* grid,
                                                            int64_t* base, uint32_t* err) {
  __shared__ int64_t sh[kScanThreads / kWave];
  set_grids<kScanThreads>(n_sets, bbox, cell, grid, base, err, sh);
}
// More than kOneGrids sets: a thread each, the cells left in place of the
// extents' first words for a scan.  (The whole join of 40,000 polygons, one
// block / this: 600 sets 98 / 101 us, 1024 108 / 108, 2048 111 / 109, 8192
// 132 / 116, 32768 241 / 134; a million sets 17 ms / 0.6.)
__global__ void __launch_bounds__(256) k_join_grids(int64_t n_sets, int4* bbox, int cell, int4* grid, uint32_t* err) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n_sets) bbox[s].x = (int)set_grid(s, bbox, cell, grid, err);
}
constexpr int64_t kOneGrids = 1024;

// A single tile's comparison is bound by its launches, a dozen of 2 to 5 us
// each with one or two more between them; what a workgroup does in about the
// time of a launch is done by one: the extents and grids of up to kFewSets sets
// of up to kBoxRun polygons in all, and the scans of up to kOneScan counts.
constexpr int kFewSets = 256;
constexpr int kFewThreads = 1024;
__global__ void __launch_bounds__(kFewThreads) k_join_grid_few(Polys A, const Meta* metaA, const int64_t* a_off,
                                                                int64_t n_sets, int cell, int4* grid, int64_t* base,
                                                                uint32_t* err) {
  __shared__ int4 boxes[kFewSets];
  __shared__ RunLds<kFewThreads, kBoxRun> lds;
  __shared__ int64_t sh[kFewThreads / kWave];
  for (int64_t s = threadIdx.x; s < n_sets; s += kFewThreads) boxes[s] = no_extent();
  __syncthreads();
  run_extents<kFewThreads, kBoxRun>(0, A.n, metaA, a_off, n_sets, lds, [&](int64_t s, const int4& m) { add_extent(boxes + s, m); });
  __syncthreads();
  set_grids<kFewThreads>(n_sets, boxes, cell, grid, base, err, sh);
}

// out[i] = sum of the first i of in[0], in[kStride], ... for i <= n, n read
// from device memory when n_ptr is given (nothing is done when it exceeds
// `room`): block totals, then every block adds the totals before its own, or,
// of more than kSumsApart blocks, takes their sum from a scan of the totals in
// between.
__device__ __forceinline__ int64_t scan_size(int64_t n, const int64_t* n_ptr, int64_t room) {
  if (n_ptr) n = *n_ptr;
  return n > room ? -1 : n;
}
template <int kStride>
__global__ void __launch_bounds__(kScanThreads) k_scan_totals(const int32_t* in, int64_t n, const int64_t* n_ptr,
                                                              int64_t room, int64_t* sums) {
  __shared__ int64_t sh[kScanThreads / kWave];
  n = scan_size(n, n_ptr, room);
  const int64_t b0 = (int64_t)blockIdx.x * kScanBlock;
  if (b0 > n) return;
  int64_t tot = 0;
  for (int k = 0; k < kScanPer; ++k) {
    const int64_t i = b0 + k * kScanThreads + threadIdx.x;
    tot += i < n ? in[i * kStride] : 0;
  }
  int64_t total;
  block_exclusive(tot, sh, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}
// Every block reading half the totals is what a scan of them costs at 16,384
// blocks of 2048 counts (the writing pass alone / with the totals' scan: 8M
// counts 67 / 73 us, 16M 127 / 137, 32M 260 / 259, 128M 1554 / 1028).
constexpr int64_t kSumsApart = 16384;
// The blocks' totals turned into the sums before them, by one workgroup.
constexpr int kOneThreads = 1024;
__global__ void __launch_bounds__(kOneThreads) k_scan_sums(int64_t n, const int64_t* n_ptr, int64_t room, int64_t* sums) {
  __shared__ int64_t sh[kOneThreads / kWave];
  n = scan_size(n, n_ptr, room);
  const int64_t blocks = n < 0 ? 0 : n / kScanBlock + 1;
  int64_t run = 0;
  for (int64_t b0 = 0; b0 < blocks; b0 += kOneThreads * kScanPer) {
    const int64_t i0 = b0 + (int64_t)threadIdx.x * kScanPer;
    int64_t v[kScanPer], tot = 0, total;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      v[k] = i0 + k < blocks ? sums[i0 + k] : 0;
      tot += v[k];
    }
    int64_t at = run + block_exclusive<kOneThreads>(tot, sh, &total);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      if (i0 + k < blocks) sums[i0 + k] = at;
      at += v[k];
    }
    run += total;
  }
}
// kClear: `in` is zeroed behind the scan; kSummed: the totals have been scanned.
template <bool kClear, int kStride, bool kSummed>
__global__ void __launch_bounds__(kScanThreads) k_scan_write(int32_t* in, int64_t n, const int64_t* n_ptr, int64_t room,
                                                             const int64_t* sums, int64_t* out) {
  __shared__ int64_t sh[kScanThreads / kWave];
  n = scan_size(n, n_ptr, room);
  const int64_t b0 = (int64_t)blockIdx.x * kScanBlock;
  if (b0 > n) return;  // the block that holds entry n writes the total
  int64_t before;
  if (kSummed) {
    before = sums[blockIdx.x];
  } else {
    int64_t mine = 0;
    for (int64_t k = threadIdx.x; k < (int64_t)blockIdx.x; k += kScanThreads) mine += sums[k];
    block_exclusive(mine, sh, &before);
  }
  const int64_t i0 = b0 + (int64_t)threadIdx.x * kScanPer;
  int32_t v[kScanPer];
  int64_t tot = 0, total;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = i0 + k < n ? in[(i0 + k) * kStride] : 0;
    tot += v[k];
  }
  int64_t run = before + block_exclusive(tot, sh, &total);
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    if (i0 + k <= n) out[i0 + k] = run;
    if (kClear && i0 + k < n) in[(i0 + k) * kStride] = 0;
    run += v[k];
  }
}
// The whole scan by one workgroup.
constexpr int64_t kOneScan = 2 * kOneThreads * kScanPer;
template <bool kClear, int kStride>
__global__ void __launch_bounds__(kOneThreads) k_scan_one(int32_t* in, int64_t n, const int64_t* n_ptr, int64_t room,
                                                          int64_t* out) {
  __shared__ int64_t sh[kOneThreads / kWave];
  n = scan_size(n, n_ptr, room);
  int64_t run = 0;
  for (int64_t b0 = 0; b0 <= n; b0 += kOneThreads * kScanPer) {
    const int64_t i0 = b0 + (int64_t)threadIdx.x * kScanPer;
    int32_t v[kScanPer];
    int64_t tot = 0, total;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      v[k] = i0 + k < n ? in[(i0 + k) * kStride] : 0;
      tot += v[k];
    }
    int64_t at = run + block_exclusive<kOneThreads>(tot, sh, &total);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      if (i0 + k <= n) out[i0 + k] = at;
      if (kClear && i0 + k < n) in[(i0 + k) * kStride] = 0;
      at += v[k];
    }
    run += total;
  }
}
int64_t scan_scratch(int64_t n) { return n / kScanBlock + 1; }
template <bool kClear, int kStride = 1>
void launch_scan(int32_t* in, int64_t n, const int64_t* n_ptr, int64_t room, int64_t* sums, int64_t* out, hipStream_t s) {
  if (room <= kOneScan) {
    hipLaunchKernelGGL((k_scan_one<kClear, kStride>), dim3(1), dim3(kOneThreads), 0, s, in, n, n_ptr, room, out);
    return;
  }
  const dim3 g((unsigned)scan_scratch(room)), b(kScanThreads);
  hipLaunchKernelGGL(k_scan_totals<kStride>, g, b, 0, s, in, n, n_ptr, room, sums);
  if (scan_scratch(room) > kSumsApart) {
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kOneThreads), 0, s, n, n_ptr, room, sums);
    hipLaunchKernelGGL((k_scan_write<kClear, kStride, true>), g, b, 0, s, in, n, n_ptr, room, sums, out);
  } else {
    hipLaunchKernelGGL((k_scan_write<kClear, kStride, false>), g, b, 0, s, in, n, n_ptr, room, sums, out);
  }
}

// ------------------------------------------------------------------- entries
// Cells of an MBR clamped to a grid: [cx0, cx1] x [cy0, cy1] (empty if cx0 > cx1).
__device__ __forceinline__ void cell_range(const Meta& m, const int4& g, int cell, int& cx0, int& cy0, int& cx1,
                                           int& cy1) {
  cx0 = max(0, cell_of(max(m.x0, g.x), g.x, cell));
  cy0 = max(0, cell_of(max(m.y0, g.y), g.y, cell));
  cx1 = min(g.z - 1, cell_of(max(m.x1 - 1, g.x), g.x, cell));
  cy1 = min(g.w - 1, cell_of(max(m.y1 - 1, g.y), g.y, cell));
  if (m.x1 <= g.x || m.y1 <= g.y) cx1 = -1;  // wholly left of or below the grid
}

// kFill false: count the A polygons of each cell; true: fill the cell lists
// (the counts start at zero again).  Nothing when the cells (or the entries)
// exceed the room for them.
template <bool kFill>
__global__ void k_join_cells(Polys A, const Meta* metaA, const int64_t* a_off, int64_t n_sets, const int4* grid,
                             const int64_t* cell_base, int cell, int64_t cell_room, int32_t* count, const int64_t* start,
                             int64_t list_room, int32_t* list) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n_cells = cell_base[n_sets];
  if (n_cells > cell_room || (kFill && start[n_cells] > list_room)) return;
  const int64_t s = set_of_lane(a_off, n_sets, a < A.n ? a : -1);
  if (s < 0) return;
  const Meta m = load_meta(metaA, a);
  const int4 g = grid[s];
  if (meta_empty(m) || g.z == 0) return;
  int cx0, cy0, cx1, cy1;
  cell_range(m, g, cell, cx0, cy0, cx1, cy1);
  for (int cy = cy0; cy <= cy1; ++cy)
    for (int cx = cx0; cx <= cx1; ++cx) {
      const int64_t c = cell_base[s] + (int64_t)cy * g.z + cx;
      const int32_t k = atomicAdd(count + c, 1);
      if (kFill) list[start[c] + k] = (int32_t)a;
    }
}

// --------------------------------------------------------------------- pairs
struct JoinArgs {
  Polys B;
  const Meta* metaA;
  const Meta* metaB;
  const int64_t* b_off;
  int64_t n_sets;
  const int4* grid;
  const int64_t* cell_base;
  const int64_t* start;
  const int32_t* list;
  int cell;
  int64_t cell_room, list_room;
};
__device__ __forceinline__ bool join_fits(const JoinArgs& a) {
  const int64_t n_cells = a.cell_base[a.n_sets];
  return n_cells <= a.cell_room && a.start[n_cells] <= a.list_room;
}

// The A polygons of B polygon b of set s, found by a group of L lanes (lane j of it;
// every lane of the group calls with the same b): emit(k, a, keep) is called
// by all of them for every L entries, k being the place of the lane's polygon
// among those kept.  The cells of one grid row that an MBR covers stand side
// by side in the lists, so that a row of them is one run of entries.  Returns
// the polygons found.
template <int L, typename F>
__device__ __forceinline__ int join_entries(const JoinArgs& a, int64_t b, int64_t s, int j, F emit) {
  if (s < 0) return 0;
  const Meta mb = load_meta(a.metaB, b);
  const int4 g = a.grid[s];
  if (meta_empty(mb) || g.z <= 0) return 0;
  int cx0, cy0, cx1, cy1, n = 0;
  cell_range(mb, g, a.cell, cx0, cy0, cx1, cy1);
  if (cx0 > cx1) return 0;
  const int shift = lane_id() / L * L;
  for (int cy = cy0; cy <= cy1; ++cy) {
    const int64_t row = a.cell_base[s] + (int64_t)cy * g.z;
    const int64_t e1 = a.start[row + cx1 + 1];
    for (int64_t e0 = a.start[row + cx0]; e0 < e1; e0 += L) {
      const int64_t e = e0 + j;
      bool keep = false;
      int32_t p = 0;
      if (e < e1) {
        p = a.list[e];
        const Meta ma = load_meta(a.metaA, p);
        const int ix0 = max(ma.x0, mb.x0), iy0 = max(ma.y0, mb.y0);
        if (ix0 < min(ma.x1, mb.x1) && iy0 < min(ma.y1, mb.y1) && cell_of(iy0, g.y, a.cell) == cy) {
          const int64_t c = row + cell_of(ix0, g.x, a.cell);
          keep = a.start[c] <= e && e < a.start[c + 1];
        }
      }
      const uint32_t m = (uint32_t)(ballot(keep) >> shift) & ((1u << L) - 1u);
      emit(n + __popc(m & ((1u << j) - 1u)), p, keep);
      n += __popc(m);
    }
  }
  return n;
}

// Pairs of each B polygon, four lanes per polygon: counted, and the first
// kFound of them kept for the second pass (a thread per polygon that searched
// again for it took 88 + 157 us for 600,000 of 4.5 pairs each).  Joins with
// eight / four / two / one: those 600,000 290 / 268 / 276 / 272 us, a million
// polygons in as many sets, where a wave's search of its set weighs, 409 / 359 /
// 343 / 327, 4096 polygons in 64 sets 73 / 72 / 84 / 88.
constexpr int kFound = 16;
constexpr int kCountLanes = 4;
__global__ void __launch_bounds__(256) k_join_count(JoinArgs a, int32_t* b_count, int32_t* found, int32_t* cell_count,
                                                    int64_t first) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (!join_fits(a)) return;
  // the cells' counts are left at zero for the next call
  const int64_t n_cells = a.cell_base[a.n_sets];
  for (int64_t c = t; first == 0 && c < n_cells; c += (int64_t)gridDim.x * blockDim.x) cell_count[c] = 0;
  const int64_t b = first + t / kCountLanes;
  const int j = (int)(t % kCountLanes);
  const int64_t s = set_of_lane(a.b_off, a.n_sets, b < a.B.n ? b : -1);
  if (b >= a.B.n) return;
  const int n = join_entries<kCountLanes>(a, b, s, j, [&](int k, int32_t p, bool keep) {
    if (keep && k < kFound) found[b * kFound + k] = p;
  });
  if (j == 0) b_count[b] = n;
}

// Each B polygon's pairs in the order of A, 16 lanes per polygon: the place of
// a pair is the number of smaller indices.  The last thread also leaves the
// sizes for the host, and the first ones the sets' offsets.
__global__ void __launch_bounds__(256) k_join_write(JoinArgs a, const int32_t* b_count, const int64_t* b_start,
                                                    const int32_t* found, int64_t cap, int32_t* out_pa, int32_t* out_pb,
                                                    int64_t* out_set_off, int64_t* sizes, int64_t first) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n_cells = a.cell_base[a.n_sets];
  const bool fits = join_fits(a);
  if (t == 0 && first == 0) {  // in host memory
    sizes[0] = n_cells;
    sizes[1] = n_cells <= a.cell_room ? a.start[n_cells] : 0;
    sizes[2] = fits ? b_start[a.B.n] : 0;
    __threadfence_system();
  }
  if (!fits) return;
  if (first == 0 && t <= a.n_sets) out_set_off[t] = b_start[min(max(a.b_off[t], (int64_t)0), a.B.n)];
  if (b_start[a.B.n] > cap) return;
  const int64_t b = first + t / kFound;
  const int j = (int)(t % kFound);
  if (b >= a.B.n) return;
  const int n = b_count[b];
  const int64_t base = b_start[b];
  if (n <= kFound) {
    const int v = j < n ? found[b * kFound + j] : INT_MAX;
    int rank = 0;
#define SCCG_RANK(R) rank += __builtin_amdgcn_update_dpp(0, v, 0x120 + R, 0xf, 0xf, false) < v ? 1 : 0;  // row_ror:R
    SCCG_RANK(1) SCCG_RANK(2) SCCG_RANK(3) SCCG_RANK(4) SCCG_RANK(5) SCCG_RANK(6) SCCG_RANK(7) SCCG_RANK(8)
    SCCG_RANK(9) SCCG_RANK(10) SCCG_RANK(11) SCCG_RANK(12) SCCG_RANK(13) SCCG_RANK(14) SCCG_RANK(15)
#undef SCCG_RANK
    if (j < n) {
      out_pa[base + rank] = v;
      out_pb[base + rank] = (int32_t)b;
    }
    return;
  }
  // more than were kept: searched again, unordered into out_pa, ordered into
  // out_pb, and back
  join_entries<kFound>(a, b, set_of(a.b_off, a.n_sets, b), j, [&](int k, int32_t p, bool keep) {
    if (keep) out_pa[base + k] = p;
  });
  __threadfence_block();
  for (int i = j; i < n; i += kFound) {
    const int32_t v = out_pa[base + i];
    int rank = 0;
    for (int k = 0; k < n; ++k) rank += out_pa[base + k] < v ? 1 : 0;
    out_pb[base + rank] = v;
  }
  __threadfence_block();
  for (int i = j; i < n; i += kFound) out_pa[base + i] = out_pb[base + i];
  __threadfence_block();
  for (int i = j; i < n; i += kFound) out_pb[base + i] = (int32_t)b;
}

static unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_join(const JoinLaunch& l, hipStream_t s) {
  const Polys &A = l.A, &B = l.B;
  if (A.n <= kBoxRun && l.n_sets <= kFewSets) {
    hipLaunchKernelGGL(k_join_grid_few, dim3(1), dim3(kFewThreads), 0, s, A, l.metaA, l.a_off, l.n_sets, l.cell, l.grid,
                       l.cell_base, l.err);
  } else {
    hipLaunchKernelGGL(k_join_init_sets, dim3(blocks_for(l.n_sets)), dim3(256), 0, s, l.n_sets, l.bbox);
    if (A.n > 0 && A.n < kSmallSets * l.n_sets)
      hipLaunchKernelGGL(k_join_bbox<kSmallRun>, dim3((unsigned)((A.n + kSmallRun - 1) / kSmallRun)), dim3(256), 0, s, A,
                         l.metaA, l.a_off, l.n_sets, l.bbox);
    else if (A.n > 0)
      hipLaunchKernelGGL(k_join_bbox<kBoxRun>, dim3((unsigned)((A.n + kBoxRun - 1) / kBoxRun)), dim3(256), 0, s, A,
                         l.metaA, l.a_off, l.n_sets, l.bbox);
    if (l.n_sets <= kOneGrids) {
      hipLaunchKernelGGL(k_join_grid, dim3(1), dim3(kScanThreads), 0, s, l.n_sets, l.bbox, l.cell, l.grid, l.cell_base,
                         l.err);
    } else {
      hipLaunchKernelGGL(k_join_grids, dim3(blocks_for(l.n_sets)), dim3(256), 0, s, l.n_sets, l.bbox, l.cell, l.grid, l.err);
      launch_scan<false, 4>(reinterpret_cast<int32_t*>(l.bbox), l.n_sets, nullptr, l.n_sets, l.sums, l.cell_base, s);
    }
  }
  if (A.n > 0)
    hipLaunchKernelGGL(k_join_cells<false>, dim3(blocks_for(A.n)), dim3(256), 0, s, A, l.metaA, l.a_off, l.n_sets,
                       l.grid, l.cell_base, l.cell, l.cell_room, l.count, nullptr, 0, nullptr);
  launch_scan<true>(l.count, 0, l.cell_base + l.n_sets, l.cell_room, l.sums, l.start, s);
  if (A.n > 0)
    hipLaunchKernelGGL(k_join_cells<true>, dim3(blocks_for(A.n)), dim3(256), 0, s, A, l.metaA, l.a_off, l.n_sets, l.grid,
                       l.cell_base, l.cell, l.cell_room, l.count, l.start, l.list_room, l.list);
  const JoinArgs j{B, l.metaA, l.metaB, l.b_off, l.n_sets, l.grid, l.cell_base, l.start, l.list, l.cell, l.cell_room,
                   l.list_room};
  for_slices(B.n, 256 / kCountLanes, [&](int64_t first, unsigned blocks) {
    hipLaunchKernelGGL(k_join_count, dim3(blocks), dim3(256), 0, s, j, l.b_count, l.found, l.count, first);
  });
  launch_scan<false>(l.b_count, B.n, nullptr, B.n, l.sums, l.b_start, s);
  for_slices(B.n, 256 / kFound, [&](int64_t first, unsigned blocks) {
    if (first == 0) blocks = std::max(blocks, blocks_for(l.n_sets + 1));
    hipLaunchKernelGGL(k_join_write, dim3(blocks), dim3(256), 0, s, j, l.b_count, l.b_start, l.found, l.cap, l.out_pa,
                       l.out_pb, l.out_set_off, l.sizes, first);
  });
  return hipGetLastError();
}
int64_t join_found_room(int64_t n_b) { return n_b * kFound; }

}  // namespace sccg
