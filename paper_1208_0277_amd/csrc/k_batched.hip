// BATCHED mode: every pair of a call in three launches, the union sweep, the
// medium sweep with the long pairs, and the persistent kernel.
//
// The method is PixelBox (Section 3): a pair box is split into sampling
// boxes, each box is classified against both polygons with Lemma 1 (open-
// interior reading: a box hovers iff an edge meets its open interior,
// otherwise its first pixel decides), boxes inside both polygons count at
// once, boxes outside either are dropped, the rest are split again, and boxes
// that fit one leaf tile are pixelized with the even-odd crossing rule.
//
// How it is laid out on gfx950 (wave64, 256 CUs in 8 XCDs):
//   - A pair box that fits one 64x64 leaf tile (the small pairs, most of any
//     pathology workload) is pixelized at once: it is below the pixelization
//     threshold T = 64*64, the n^2 end of Section 3.4's range for n = 64.
//     When even the union of the two MBRs fits one tile, that tile is used
//     and I and U are both counted there, so the ring areas are not needed
//     (SCCG_F_NO_UNION_TILE turns this off).
//   - Larger boxes are split into at most 8x8 cells whose side is 64*8^l, so
//     that every split lands on leaf tiles after l more levels.  One wave
//     classifies all cells of a box in one pass over the edges: each lane
//     takes one edge and sets the bits of the cells it hovers and of the
//     cells whose first pixel it crosses, in two 64-bit masks, which are then
//     OR- and XOR-reduced across the wave.  Cost O(edges) per split instead of
//     O(cells x edges).  A split into fewer than min_classify_cells leaf
//     tiles is not classified: its tiles are pixelized directly.
//   - Rings are read 64 vertices at a time with the next chunk in flight
//     (RingStream); a vertex's successor comes from the next lane.
//   - Leaf tiles use bit-sliced crossing tests: a lane holds one column of
//     the tile as a row mask.  Each vertical edge of the tile's band XORs its
//     row mask into the LDS slot of the rightmost column it toggles (one
//     atomic per edge), and a prefix XOR over the lanes turns the slots into
//     every column's crossing parities.  A polygon known to contain a tile
//     is not tested again (its mask is all ones).  When a split leaves
//     several leaf tiles, each ring is streamed once per band row, its edges
//     scattered into the slots of the row's columns in LDS, and the tiles of
//     the row are scanned from those, right to left.
//   - The pair's MBRs and shoelace areas are reduced by the wave that takes
//     the pair, from the same coalesced ring loads it needs anyway; the
//     pairs with many vertices ("long", claimed first: a largest-first
//     order) get them from two waves, one per ring, which count the pair at
//     once unless its box has more than 64 leaf tiles: then any wave of the
//     persistent kernel can take one of its boxes.
//   - The sweeps share their pairs out statically; the persistent grid's
//     waves claim, in this order: boxes from their queue, listed pairs, boxes
//     from any queue.  Claims go through per-stream counters (one stream per
//     XCD) on cache lines of their own, and so do the appends to the lists: a
//     counter takes an atomic every 7 ns.  A listed pair's split publishes its
//     continuing boxes to a device queue when there are enough of them, so that idle
//     waves share the pair.  Queue slots are single 64-bit words written and
//     taken with atomics, so no cache flushes are needed; a consumer that
//     overshoots the tail marks the slot skipped and the producer keeps that
//     box, so every box is processed exactly once and nobody waits on work
//     that may never come.  The one remaining wait (a slot reserved but not
//     yet written) is on a producer that writes right after reserving; it is
//     bounded anyway and latches SCCG_E_DEVICE if the bound is hit.
#include <limits.h>
#include <stddef.h>

#include <algorithm>

#include <type_traits>

#include "sccg_device.h"

namespace sccg {

constexpr int kLocalCap = 256;          // per-wave stack of boxes to process inline
constexpr uint32_t kSpinLimit = 1u << 22;
// per-wave LDS of the persistent kernel: the slots of one band row of each
// ring (a single tile's leaf slots are the first of them), the inline box
// stack
constexpr int kRowSlotsPerWave = 2 * kMaxGrid * kWave;
constexpr int kLdsPerWave = kRowSlotsPerWave * 8 + kLocalCap * 8;
constexpr unsigned long long kSkip = 1ull;  // slot abandoned by an overshooting consumer

int batch_lds_bytes_per_wave() { return kLdsPerWave; }

// ---------------------------------------------------------------- task words
// [63] valid | [56:55] level | [54] p inside | [53] q inside | [52:44] ty |
// [43:35] tx | [30:0] heavy-list index.  tx, ty: cell origin in 64-px units
// from the pair-box origin; level l: cell side 64 * 8^l (0 = leaf tile).
__device__ __forceinline__ uint64_t task_word(int64_t hidx, int level, int tx, int ty, bool kp, bool kq) {
  return (1ull << 63) | ((uint64_t)level << 55) | ((uint64_t)kp << 54) | ((uint64_t)kq << 53) |
         ((uint64_t)ty << 44) | ((uint64_t)tx << 35) | (uint64_t)hidx;
}
struct Task {
  int64_t hidx;
  int level, tx, ty;
  bool kp, kq;
};
__device__ __forceinline__ Task task_decode(uint64_t w) {
  Task t;
  t.hidx = (int64_t)(w & 0x7fffffffull);
  t.tx = (int)((w >> 35) & 0x1ff);
  t.ty = (int)((w >> 44) & 0x1ff);
  t.kq = (w >> 53) & 1;
  t.kp = (w >> 54) & 1;
  t.level = (int)((w >> 55) & 3);
  return t;
}

// ------------------------------------------------------------- bit helpers
// cell (i, j) of an 8x8 grid is bit 8*j + i
__device__ __forceinline__ uint64_t rows_bits(int j0, int j1) {
  return (~0ull >> (8 * (7 - j1))) & (~0ull << (8 * j0));
}
__device__ __forceinline__ uint64_t spread(uint32_t colbyte) { return (uint64_t)colbyte * 0x0101010101010101ull; }
__device__ __forceinline__ uint32_t cols_bits(int i0, int i1) { return (0xFFu >> (7 - i1)) & (0xFFu << i0) & 0xFFu; }
// rows [lo, hi) of a 64-row tile, 0 <= lo < hi <= 64
__device__ __forceinline__ uint64_t row_range(int lo, int hi) {
  return (~0ull << lo) & (~0ull >> (64 - hi));
}
// x limited to [lo, hi]: a coordinate clamped to a box's sides before the
// box origin is subtracted, since |x| <= 2^30 on both sides of a difference
// could leave int32
__device__ __forceinline__ int clamp_to(int x, int lo, int hi) { return min(max(x, lo), hi); }

// ----------------------------------------------------------------- context
struct Ctx {
  const BatchArgs* a;
  bool stats;       // work counters on (a compile-time false in the sweeps' plain instances)
  int lane;
  uint64_t* slots;  // per-wave leaf slots
  uint64_t* local;  // per-wave inline stack, kLocalCap entries
  int lsp;          // inline stack depth (wave-uniform)
  int home;         // preferred queue
  int xcd;          // first claim stream (the workgroup's XCD under round-robin dispatch)
};

// Work counters (only with sccg_set_stats): one atomic per event from lane 0.
// The first stream at or after `from` (cyclically, kStreams of them) not in
// the exhausted mask `empty` (wave-uniform; at least one must be left).
__device__ __forceinline__ int next_stream(uint32_t empty, int from) {
  const uint32_t avail = ~empty & ((1u << kStreams) - 1u);
  const uint32_t rot = ((avail >> from) | (avail << (kStreams - from))) & ((1u << kStreams) - 1u);
  return uniform((from + __ffs((int)rot) - 1) % kStreams);
}

// Stamp of the device's constant-rate counter (100 MHz), read by the wave.
__device__ __forceinline__ unsigned long long wave_stamp(const BatchArgs& a) {
  return a.wave_t ? (unsigned long long)__builtin_amdgcn_s_memrealtime() : 0ull;
}
// A wave's (start, end) stamps of kernel `kernel` (see BatchArgs::wave_t).
__device__ __forceinline__ void wave_stamps(const BatchArgs& a, int kernel, unsigned long long t0, int lane) {
  if (!a.wave_t || lane != 0) return;
  const unsigned w = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (w >= (unsigned)a.wave_cap) return;
  unsigned long long* p = a.wave_t + 2 * ((size_t)kernel * (size_t)a.wave_cap + w);
  p[0] = t0;
  p[1] = (unsigned long long)__builtin_amdgcn_s_memrealtime();
}

__device__ __forceinline__ void stat_add(const Ctx& c, int k, unsigned long long v) {
  if (c.stats && c.lane == 0 && v) atomicAdd(&c.a->st->stats[k], v);
}

// What a wave needs to work on one pair.
struct PairInfo {
  int64_t pair;     // index into the pair arrays
  int64_t hidx;     // heavy-list index, or -1 when the pair is not shared
  int64_t op, np, oq, nq;
  Meta box;
  int64_t area_sum;  // |p| + |q|
};

// PairInfo fields are wave-uniform: keep them in scalar registers.
__device__ __forceinline__ void make_uniform(PairInfo& pi) {
  pi.pair = uniform64(pi.pair);
  pi.hidx = uniform64(pi.hidx);
  pi.op = uniform64(pi.op);
  pi.np = uniform64(pi.np);
  pi.oq = uniform64(pi.oq);
  pi.nq = uniform64(pi.nq);
  pi.box.x0 = uniform(pi.box.x0);
  pi.box.y0 = uniform(pi.box.y0);
  pi.box.x1 = uniform(pi.box.x1);
  pi.box.y1 = uniform(pi.box.y1);
  pi.area_sum = uniform64(pi.area_sum);
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------- ring scans
// The value of the next lane (DPP wave shift left by one; lane 63 reads 0).
__device__ __forceinline__ int2 next_lane(int2 v) {
  return make_int2(__builtin_amdgcn_update_dpp(0, v.x, 0x130, 0xf, 0xf, false),
                   __builtin_amdgcn_update_dpp(0, v.y, 0x130, 0xf, 0xf, false));
}

__device__ __forceinline__ int2 lane_value(int2 v, int l) {
  return make_int2(__builtin_amdgcn_readlane(v.x, l), __builtin_amdgcn_readlane(v.y, l));
}

// A ring read 64 vertices at a time with loads running ahead: lane L holds
// vertex base + L in `cur` and vertex base + 64 + L in `nxt`; ahead(), called
// at the top of each iteration, starts the load of the chunk after `nxt`, so
// that it arrives while the current chunk is processed.  A vertex's
// successor is the next lane's vertex; lane 63's is lane 0 of `nxt`, and the
// last vertex's is the first.  `nv` (>= 1) must be wave-uniform.  Lanes past the end load the
// last vertex again (the index is clamped, so the loads need no branch) and
// must be masked with valid(): the successor shift reads across lanes, so
// no lane may be switched off around it, and a per-lane branch in the loop
// body lets the compiler split the wave.
struct RingStream {
  const int2* p;
  int nv, base, lane;
  int2 first, cur, nxt, nn;

  __device__ __forceinline__ int2 at(int k) const { return p[min(k, nv - 1)]; }
  __device__ __forceinline__ RingStream(const int2* xy, int64_t o, int nv_, int lane_, int base0 = 0,
                                        const int2* first_ = nullptr)
      : p(xy + o), nv(uniform(nv_)), base(uniform(base0)), lane(lane_) {
    cur = at(base + lane);
    nxt = at(base + kWave + lane);
    first = first_ ? *first_ : lane_value(cur, 0);
  }
  __device__ __forceinline__ void ahead() { nn = at(base + 2 * kWave + lane); }
  __device__ __forceinline__ bool valid() const { return base + lane < nv; }
  // successor of this lane's vertex (every lane takes part)
  __device__ __forceinline__ int2 succ() const {
    const int2 s = next_lane(cur);
    const int2 n0 = lane_value(nxt, 0);
    const bool wrap = base + lane + 1 == nv, last = lane == kWave - 1;
    return make_int2(wrap ? first.x : (last ? n0.x : s.x), wrap ? first.y : (last ? n0.y : s.y));
  }
  __device__ __forceinline__ bool next() {
    base = uniform(base + kWave);
    if (base >= nv) return false;
    cur = nxt;
    nxt = nn;
    return true;
  }
};

// The ablations of Section 5.2 (SCCG_F_PIXEL_ONLY, SCCG_F_NO_SEP) count the
// union directly, over the bounding box of both MBRs, instead of deriving it
// from the areas.  Counts of one box then travel packed: intersection in
// the low 32 bits, direct union in the high 32 (a processed box has at most
// 32767^2 < 2^32 pixels).
__device__ __forceinline__ bool direct_union(const BatchArgs& a) {
  return (a.flags & (SCCG_F_PIXEL_ONLY | SCCG_F_NO_SEP)) != 0u;
}

// Wave total of a lane's intersection count n and, when `direct`, of its
// union count nu, packed.
__device__ __forceinline__ uint64_t pack_counts(uint32_t n, uint32_t nu, bool direct) {
  if (!direct) return wave_sum_u32(n);
  // a lane holds at most 64 pixels of each, so both wave sums stay below
  // 2^13 and travel in the two halves of one 32-bit sum
  const uint32_t t = wave_sum_u32(n | (nu << 16));
  return (uint64_t)(t & 0xffffu) | ((uint64_t)(t >> 16) << 32);
}

// ------------------------------------------------------------------ leaves
// Scatter-and-scan leaves.  The columns of a leaf tile live in lanes in
// reverse order: in a W-column group (W = 64, or 32 when p and q share the
// wave as two halves), lane L holds column W - 1 - L.  A vertical edge at X
// whose span meets the tile's rows toggles those rows in every column left of
// X.  It XORs its row mask into one LDS slot: the slot of the rightmost column
// it toggles, W - min(X - x0, W).  Any number of edges may share a slot.  An
// inclusive prefix XOR over the lanes then leaves in every column the XOR of
// the edges right of it: bit r of lane L is the crossing parity of the centre
// of pixel (x0 + W - 1 - L, y0 + r) (Section 3.1).  Cost per tile: one atomic
// per edge of the band, no per-edge work in the other lanes.

// Inclusive prefix XOR over lanes (rows of 16 by shifts, then the row
// broadcasts); with kHalves the scan restarts at lane 32.
template <bool kHalves>
__device__ __forceinline__ uint32_t wave_prefix_xor(uint32_t x) {
  x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  if (!kHalves) x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return x;
}
template <bool kHalves>
__device__ __forceinline__ uint64_t wave_prefix_xor(uint64_t x) {
  return ((uint64_t)wave_prefix_xor<kHalves>((uint32_t)(x >> 32)) << 32) | wave_prefix_xor<kHalves>((uint32_t)x);
}

// The slot and row mask of edge (v, w) for the tile at (tx0, ty0) of height
// th in a W-column group: kept iff vertical, right of the tile's left side,
// with a span meeting the rows.
__device__ __forceinline__ bool leaf_edge(int2 v, int2 w, int tx0, int ty0, int th, int W, int& slot,
                                          uint64_t& rr) {
  if (v.x != w.x) return false;
  const int lo = clamp_to(min(v.y, w.y), ty0, ty0 + th) - ty0;
  const int hi = clamp_to(max(v.y, w.y), ty0, ty0 + th) - ty0;
  const int dx = min(v.x, tx0 + W) - tx0;
  if (!(lo < hi && dx > 0)) return false;
  slot = W - dx;
  rr = row_range(lo, hi);
  return true;
}

template <typename M>
__device__ __forceinline__ void slot_xor(M* slots, int k, uint64_t rr) {
  __hip_atomic_fetch_xor(slots + k, (M)rr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Scatter the leaf edges of one ring into slots[base ..).  Edges right of the
// whole group (they toggle every column) are XORed into *full (per lane)
// instead of slot 0, so that they do not all hit one LDS address.
__device__ __forceinline__ void scatter_ring(Ctx& c, const int2* xy, int64_t o, int64_t nv, int tx0, int ty0, int th,
                                             int W, uint64_t* slots, int base, uint64_t* full) {
  const int n = uniform((int)nv);
  uint32_t kept = 0;
  if (n > 0) {
    RingStream rs(xy, o, n, c.lane);
#pragma unroll 1
    do {
      rs.ahead();
      const int2 w = rs.succ();
      int slot = 0;
      uint64_t rr = 0;
      const bool keep = rs.valid() && leaf_edge(rs.cur, w, tx0, ty0, th, W, slot, rr);
      if (keep) {
        if (slot == 0)
          *full ^= rr;
        else
          slot_xor(slots, base + slot, rr);
      }
      if (c.stats) kept += (uint32_t)__popcll(ballot(keep));
    } while (rs.next());
  }
  if (c.stats) {
    stat_add(c, 8, (unsigned long long)kept);
    stat_add(c, 10, (unsigned long long)nv);
  }
}

// Zero for clearing leaf slots, made where it is stored: a zero the compiler
// hoists into a long-lived register pair gets spilled to scratch under this
// kernel's register pressure.
template <typename M>
__device__ __forceinline__ M fresh_zero() {
  uint32_t lo, hi;
  asm volatile("v_mov_b32 %0, 0" : "=v"(lo));
  if (sizeof(M) == 4) return (M)lo;
  asm volatile("v_mov_b32 %0, 0" : "=v"(hi));
  return (M)(((uint64_t)hi << 32) | lo);
}

// Pixels of the tile [tx0, tx0+tw) x [ty0, ty0+th) inside both polygons; a
// polygon known to contain the tile is not scattered (all rows set).
__device__ __forceinline__ uint64_t leaf_count(Ctx& c, const PairInfo& pi, int tx0, int ty0, int tw, int th, bool kp,
                                               bool kq) {
  const BatchArgs& a = *c.a;
  const int lane = c.lane;
  uint64_t* slots = c.slots;
  slots[lane] = fresh_zero<uint64_t>();
  slots[kWave + lane] = fresh_zero<uint64_t>();
  wave_sync_lds();
  uint64_t fp = 0, fq = 0;
  if (!kp) scatter_ring(c, a.A.xy, pi.op, pi.np, tx0, ty0, th, kWave, slots, 0, &fp);
  if (!kq) scatter_ring(c, a.B.xy, pi.oq, pi.nq, tx0, ty0, th, kWave, slots, kWave, &fq);
  wave_sync_lds();
  const uint64_t full = row_range(0, th);
  const uint64_t mp = kp ? full : wave_prefix_xor<false>(slots[lane]) ^ wave_xor64(fp);
  const uint64_t mq = kq ? full : wave_prefix_xor<false>(slots[kWave + lane]) ^ wave_xor64(fq);
  wave_sync_lds();
  const bool in_tile = kWave - 1 - lane < tw;
  const uint32_t n = in_tile ? (uint32_t)__popcll(mp & mq) : 0u;
  const uint32_t nu = in_tile ? (uint32_t)__popcll(mp | mq) : 0u;
  if (c.stats) {
    stat_add(c, 1, 1ull);
    stat_add(c, 0, (unsigned long long)tw * th * ((kp ? 0 : 1) + (kq ? 0 : 1)));
  }
  return pack_counts(n, nu, direct_union(a));
}

// Row-wide leaves.  When a split leaves several leaf tiles, each band row of
// it (up to kMaxGrid tiles) is pixelized at once: one slot array per ring
// holds every column of the row, position Wpad - 1 - (column - bx0) for
// Wpad = 64 x (tiles per row), so that a vertical edge at X toggles the
// positions from Wpad - min(X - bx0, Wpad) up, with one atomic whatever its
// distance.  Each ring is streamed once per band row (from L2: its pair's
// rings were read moments before).  Inside each tile's block of 64 positions
// a prefix XOR over the lanes gives the tile's columns their crossing
// parities for the edges that end inside it; the blocks of the tiles to its
// right add the XOR of all their slots, carried from block to block.
constexpr int kRowSlots = kMaxGrid * kWave;  // slots of one ring's band row

// Scatter the vertical edges of one ring that meet rows [ry0, ry0 + th) into
// a row's slots (wpad positions from bx0).
__device__ __forceinline__ void scatter_row(Ctx& c, const int2* xy, int64_t o, int64_t nv, int bx0, int wpad, int ry0,
                                            int th, uint64_t* slots) {
  const int n = uniform((int)nv);
  if (n <= 0) return;
  uint32_t kept = 0;
  RingStream rs(xy, o, n, c.lane);
#pragma unroll 1
  do {
    rs.ahead();
    const int2 w = rs.succ();
    int slot = 0;
    uint64_t rr = 0;
    const bool keep = rs.valid() && leaf_edge(rs.cur, w, bx0, ry0, th, wpad, slot, rr);
    if (keep) slot_xor(slots, slot, rr);
    if (c.stats) kept += (uint32_t)__popcll(ballot(keep));
  } while (rs.next());
  if (c.stats) {
    stat_add(c, 8, (unsigned long long)kept);
    stat_add(c, 10, (unsigned long long)n);
  }
}

// The leaf tiles `cont` (bit 8j + i = tile (i, j) of side 64 from (bx0, by0))
// of a split.  kin_p / kin_q: tiles known to lie inside p / q.  A lone tile
// is scattered straight from the rings; otherwise a band row at a time.
__device__ __forceinline__ void leaf_rows(Ctx& c, const PairInfo& pi, int bx0, int by0, int bx1, int by1, int gy,
                                          uint64_t cont, uint64_t kin_p, uint64_t kin_q, uint64_t& acc) {
  const BatchArgs& a = *c.a;
  if (__popcll(cont) == 1) {
    const int t = __ffsll((long long)cont) - 1, i = t & 7, j = t >> 3;
    const int tx0 = bx0 + kTile * i, ty0 = by0 + kTile * j;
    acc += leaf_count(c, pi, tx0, ty0, min(kTile, bx1 - tx0), min(kTile, by1 - ty0), (kin_p >> t) & 1ull,
                      (kin_q >> t) & 1ull);
    return;
  }
  const int lane = c.lane;
  const bool direct = direct_union(a);
  const int gx = uniform((bx1 - bx0 + kTile - 1) / kTile);
  const int wpad = gx * kTile;
  uint64_t* sp = c.slots;
  uint64_t* sq = c.slots + kRowSlots;
  uint32_t ni = 0, nu = 0;  // this lane's pixels counted, over every tile
  unsigned long long n_leaf = 0, n_tests = 0;
#pragma unroll 1
  for (int j = 0; j < gy; ++j) {
    const uint32_t row = (uint32_t)(cont >> (8 * j)) & 0xffu;
    if (!row) continue;
    const uint32_t kp_row = (uint32_t)(kin_p >> (8 * j)) & row, kq_row = (uint32_t)(kin_q >> (8 * j)) & row;
    const bool need_p = kp_row != row, need_q = kq_row != row;
    const int ry0 = by0 + kTile * j, th = min(kTile, by1 - ry0);
    const uint64_t full = row_range(0, th);
#pragma unroll 1
    for (int b = 0; b < gx; ++b) {
      sp[b * kWave + lane] = fresh_zero<uint64_t>();
      sq[b * kWave + lane] = fresh_zero<uint64_t>();
    }
    wave_sync_lds();
    if (need_p) scatter_row(c, a.A.xy, pi.op, pi.np, bx0, wpad, ry0, th, sp);
    if (need_q) scatter_row(c, a.B.xy, pi.oq, pi.nq, bx0, wpad, ry0, th, sq);
    wave_sync_lds();
    // tiles right to left: block b = gx - 1 - i holds tile i
    uint64_t carry_p = 0, carry_q = 0;
#pragma unroll 1
    for (int i = gx - 1; i >= 0; --i) {
      const int b = gx - 1 - i;
      const uint64_t xp = wave_prefix_xor<false>(sp[b * kWave + lane]);
      const uint64_t xq = wave_prefix_xor<false>(sq[b * kWave + lane]);
      if ((row >> i) & 1u) {
        const int tw = min(kTile, bx1 - (bx0 + kTile * i));
        const uint64_t mp = ((kp_row >> i) & 1u) ? full : (xp ^ carry_p);
        const uint64_t mq = ((kq_row >> i) & 1u) ? full : (xq ^ carry_q);
        if (kWave - 1 - lane < tw) {
          ni += (uint32_t)__popcll(mp & mq);
          nu += (uint32_t)__popcll(mp | mq);
        }
        n_leaf += 1;
        n_tests += (unsigned long long)tw * th * ((((kp_row >> i) & 1u) ? 0 : 1) + (((kq_row >> i) & 1u) ? 0 : 1));
      }
      carry_p ^= (uint64_t)readlane64((int64_t)xp, kWave - 1);
      carry_q ^= (uint64_t)readlane64((int64_t)xq, kWave - 1);
    }
    wave_sync_lds();
  }
  const uint64_t si = wave_sum_u32(ni);
  acc += direct ? (si | ((uint64_t)wave_sum_u32(nu) << 32)) : si;
  if (c.stats) {
    stat_add(c, 1, n_leaf);
    stat_add(c, 0, n_tests);
  }
}

// One pass over the ring: hover mask H and first-pixel parity mask P of the
// gx x gy cells of side 2^ls covering [bx0,bx1) x [by0,by1).
__device__ __forceinline__ void classify(Ctx& c, const int2* xy, int64_t o, int64_t nv, int bx0, int by0, int bx1, int by1, int ls,
                         int gx, int gy, uint64_t& H, uint64_t& P) {
  const int S = 1 << ls;
  uint64_t h = 0, p = 0;
  if (uniform((int)nv) <= 0) {
    H = 0;
    P = 0;
    return;
  }
  RingStream rs(xy, o, uniform((int)nv), c.lane);
#pragma unroll 1
  do {
    rs.ahead();
    const int2 v = rs.cur, w = rs.succ();
    if (!rs.valid()) {
      // past the end of the ring
    } else if (v.x == w.x) {
      // coordinates past the box's far sides are clamped to them (the tests
      // below do not change), so that no difference leaves int32
      const int X = min(v.x, bx1), lo = min(min(v.y, w.y), by1), hi = min(max(v.y, w.y), by1);
      const int dx = X - bx0;
      if (dx > 0 && hi > by0) {
        // hover: X strictly inside a column, span meeting the open rows
        if (X < bx1 && (dx & (S - 1)) != 0 && lo < by1) {
          const int i = dx >> ls;
          const int j0 = lo > by0 ? (lo - by0) >> ls : 0;
          const int j1 = min(gy - 1, ((hi - by0 + S - 1) >> ls) - 1);
          if (j0 <= j1) h |= rows_bits(j0, j1) & spread(1u << i);
        }
        // crossing of the first pixel (c_i, r_j) of cells with c_i < X, lo <= r_j < hi
        const int ic = min(gx - 1, ((dx + S - 1) >> ls) - 1);
        const int ja = lo > by0 ? ((lo - by0 + S - 1) >> ls) : 0;
        const int jb = min(gy - 1, ((hi - by0 + S - 1) >> ls) - 1);
        if (ja <= jb) p ^= rows_bits(ja, jb) & spread(0xFFu >> (7 - ic));
      }
    } else {
      const int Y = min(v.y, by1), lo = min(min(v.x, w.x), bx1), hi = min(max(v.x, w.x), bx1);
      const int dy = Y - by0;
      if (dy > 0 && Y < by1 && (dy & (S - 1)) != 0 && lo < bx1 && hi > bx0) {
        const int j = dy >> ls;
        const int i0 = lo > bx0 ? (lo - bx0) >> ls : 0;
        const int i1 = min(gx - 1, ((hi - bx0 + S - 1) >> ls) - 1);
        if (i0 <= i1) h |= rows_bits(j, j) & spread(cols_bits(i0, i1));
      }
    }
  } while (rs.next());
  H = wave_or64(h);
  P = wave_xor64(p);
  stat_add(c, 9, (unsigned long long)nv);
}

// Add a shared pair's partial counts: `n` packed as by pack_counts.  The
// union starts at |p| + |q| and loses every intersection pixel, or (direct
// union) starts at 0 and gains every union pixel.
__device__ __forceinline__ void add_counts(const BatchArgs& a, int64_t pair, uint64_t n) {
  if (n == 0) return;
  const unsigned long long i = n & 0xffffffffull;
  const unsigned long long u = direct_union(a) ? (n >> 32) : (0 - i);
  if (i) atomicAdd(reinterpret_cast<unsigned long long*>(a.inter + pair), i);
  if (u) atomicAdd(reinterpret_cast<unsigned long long*>(a.uni + pair), u);
}

// ------------------------------------------------------------------- queue
// Queue q is a head counter, a tail counter and queue_cap slots.  A producer
// reserves slots with one atomic add on the tail and fills each with a
// compare-and-swap from 0; a consumer takes a ticket with one atomic add on
// the head.  A ticket below the tail is a reserved slot: the consumer waits
// for its word.  A ticket at or past the tail tries to mark its slot skipped;
// if it wins, the producer that later reserves the slot finds it taken and
// keeps the box; if it loses, the word is there and the consumer takes it.
__device__ __forceinline__ bool queue_claim_one(Ctx& c, int q, uint64_t* out) {
  const BatchArgs& a = *c.a;
  uint64_t word = 0;
  if (c.lane == 0) {
    unsigned long long* head = &a.st->q_head[q].v;
    unsigned long long* tail = &a.st->q_tail[q].v;
    const unsigned long long cap = (unsigned long long)a.queue_cap;
    const unsigned long long h0 = __hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long t = __hip_atomic_load(tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (h0 < cap && h0 < t) {
      const unsigned long long h = atomicAdd(head, 1ull);
      if (h < cap) {
        unsigned long long* slot = a.queue + (size_t)q * a.queue_cap + h;
        t = __hip_atomic_load(tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (h < t) {
          uint32_t spins = 0;
          while ((word = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
            if (++spins > kSpinLimit) {
              latch_error(a.err, kErrWatchdog);
              break;
            }
            __builtin_amdgcn_s_sleep(1);
          }
        } else {
          const unsigned long long prev = atomicCAS(slot, 0ull, kSkip);
          word = (prev == 0ull) ? 0ull : prev;
        }
        if (word == kSkip) word = 0;
      }
    }
  }
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)word, 0, kWave);
  const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(word >> 32), 0, kWave);
  *out = ((uint64_t)hi << 32) | lo;
  return *out != 0;
}

// Claim from the home queue only, or from every queue (home first).
__device__ __forceinline__ bool queue_claim(Ctx& c, bool all, uint64_t* out) {
  const int nq = all ? c.a->n_queues : 1;
  for (int r = 0; r < nq; ++r)
    if (queue_claim_one(c, (c.home + r) % c.a->n_queues, out)) return true;
  return false;
}

// Children of one split: lane j (< n) holds word j.  Publish them to the
// queue when the pair is shared and there are enough, else (and for what a
// full queue or a skip-marked slot refuses) keep them on the wave's stack.
__device__ __forceinline__ void emit_children(Ctx& c, const PairInfo& pi, uint64_t word, bool has, int n) {
  const BatchArgs& a = *c.a;
  const uint64_t b = ballot(has);
  const int rank = lanes_below(b);
  bool keep = has;
  if (pi.hidx >= 0 && !(a.flags & SCCG_F_NO_SPLIT_QUEUE) && n >= a.min_cells_to_queue) {
    unsigned long long t = 0;
    if (c.lane == 0) t = atomicAdd(&a.st->q_tail[c.home].v, (unsigned long long)n);
    t = (unsigned long long)uniform64((int64_t)__shfl((long long)t, 0, kWave));
    if (has && t + rank < (unsigned long long)a.queue_cap) {
      unsigned long long* slot = a.queue + (size_t)c.home * a.queue_cap + t + rank;
      const unsigned long long prev = atomicCAS(slot, 0ull, (unsigned long long)word);
      keep = prev != 0ull;  // skip-marked: the box stays here
    }
    if (c.stats) {
      const int kept = __popcll(ballot(keep));
      stat_add(c, 3, (unsigned long long)(n - kept));
      stat_add(c, 4, (unsigned long long)kept);
    }
  }
  const uint64_t bk = ballot(keep);
  const int nk = __popcll(bk);
  if (nk > 0) {
    if (keep) c.local[c.lsp + lanes_below(bk)] = word;
    c.lsp += nk;
    wave_sync_lds();
  }
}

// Pixels of the cells `m` of a gx x gy grid of side S whose last column and
// row are lw and lh wide.
__device__ __forceinline__ uint64_t cells_area(uint64_t m, int gx, int gy, int S, int lw, int lh) {
  uint64_t add = 0;
  for (int j = 0; j < gy; ++j) {
    const uint32_t row = (uint32_t)(m >> (8 * j)) & 0xFFu;
    if (!row) continue;
    const uint64_t hgt = (j == gy - 1) ? (uint64_t)lh : (uint64_t)S;
    const uint32_t last = (row >> (gx - 1)) & 1u;
    add += hgt * ((uint64_t)(__popc(row) - last) * S + (uint64_t)last * lw);
  }
  return add;
}

// Split box [bx0,bx1) x [by0,by1) of a pair (already known to be a
// continuing box) into cells of level `cl` (side 64*8^cl).  Cells inside
// both polygons add their size to `acc`; continuing cells become tasks.
__device__ __forceinline__ void split_box(Ctx& c, const PairInfo& pi, int bx0, int by0, int bx1, int by1, int cl, bool kp, bool kq,
                          uint64_t& acc) {
  const BatchArgs& a = *c.a;
  const int ls = 6 + 3 * cl;
  const int S = 1 << ls;
  const int gx = (bx1 - bx0 + S - 1) >> ls, gy = (by1 - by0 + S - 1) >> ls;
  const uint64_t valid = rows_bits(0, gy - 1) & spread(cols_bits(0, gx - 1));
  uint64_t Hp = 0, Pp = valid, Hq = 0, Pq = valid;
  if (a.flags & SCCG_F_PIXEL_ONLY) {
    Hp = Hq = valid;  // PixelOnly: no sampling boxes, every cell is pixelized
  } else if (cl == 0 && gx * gy < a.min_classify_cells) {
    // a split into a few leaf tiles: classifying them costs two ring passes
    // and rarely decides a tile, so every tile is pixelized (a polygon known
    // to contain the box still counts as inside)
    if (!kp) Hp = valid;
    if (!kq) Hq = valid;
  } else {
    if (!kp) classify(c, a.A.xy, pi.op, pi.np, bx0, by0, bx1, by1, ls, gx, gy, Hp, Pp);
    if (!kq) classify(c, a.B.xy, pi.oq, pi.nq, bx0, by0, bx1, by1, ls, gx, gy, Hq, Pq);
  }
  const uint64_t in_p = ~Hp & Pp & valid, out_p = ~Hp & ~Pp & valid;
  const uint64_t in_q = ~Hq & Pq & valid, out_q = ~Hq & ~Pq & valid;
  const uint64_t both = in_p & in_q;
  uint64_t cont = valid & ~out_p & ~out_q & ~both;
  uint64_t uni_add = 0;  // cells that stop inside p or q (direct union only)
  if (direct_union(a)) {
    // a cell stops only when decided for the intersection (inside both, or
    // outside one) and for the union (inside one, or outside both)
    const uint64_t dec_i = both | out_p | out_q, dec_u = in_p | in_q | (out_p & out_q);
    cont = valid & ~(dec_i & dec_u);
    uni_add = (in_p | in_q) & valid & ~cont;
  }
  const int lw = (bx1 - bx0) - (gx - 1) * S, lh = (by1 - by0) - (gy - 1) * S;
  // cells inside both polygons contribute their size at once
  if (both) acc += cells_area(both, gx, gy, S, lw, lh);
  if (uni_add) acc += cells_area(uni_add, gx, gy, S, lw, lh) << 32;
  stat_add(c, 2, 1ull);
  const int n = __popcll(cont);
  // leaf tiles that this wave keeps: process them now, a band row at a time
  const bool publish = pi.hidx >= 0 && !(a.flags & SCCG_F_NO_SPLIT_QUEUE) && n >= a.min_cells_to_queue;
  if (cl == 0 && n && !publish) {
    const uint64_t kn = (a.flags & SCCG_F_NO_KNOWN_INSIDE) ? 0ull : ~0ull;
    leaf_rows(c, pi, bx0, by0, bx1, by1, gy, cont, in_p & kn, in_q & kn, acc);
    return;
  }
  // one lane per continuing cell
  bool has = false;
  uint64_t word = 0;
  if ((cont >> c.lane) & 1ull) {
    const int i = c.lane & 7, j = c.lane >> 3;
    const int tx = ((bx0 - pi.box.x0) >> 6) + (i << (3 * cl));
    const int ty = ((by0 - pi.box.y0) >> 6) + (j << (3 * cl));
    has = true;
    word = task_word(pi.hidx < 0 ? 0 : pi.hidx, cl, tx, ty, (in_p >> c.lane) & 1ull, (in_q >> c.lane) & 1ull);
  }
  if (n) emit_children(c, pi, word, has, n);
}

// Process one box task of pair `pi`: a leaf tile or a further split.
__device__ __forceinline__ void run_box(Ctx& c, const PairInfo& pi, uint64_t w, uint64_t& acc) {
  const BatchArgs& a = *c.a;
  const Task t = task_decode(w);
  const int side = kTile << (3 * t.level);
  const int x0 = pi.box.x0 + t.tx * kTile, y0 = pi.box.y0 + t.ty * kTile;
  const int x1 = min(x0 + side, pi.box.x1), y1 = min(y0 + side, pi.box.y1);
  const bool kp = t.kp && !(a.flags & SCCG_F_NO_KNOWN_INSIDE);
  const bool kq = t.kq && !(a.flags & SCCG_F_NO_KNOWN_INSIDE);
  if (t.level == 0)
    acc += leaf_count(c, pi, x0, y0, x1 - x0, y1 - y0, kp, kq);
  else
    split_box(c, pi, x0, y0, x1, y1, t.level - 1, kp, kq, acc);
}

__device__ __forceinline__ void drain_local(Ctx& c, const PairInfo& pi, uint64_t& acc) {
  while (c.lsp > 0) {
    c.lsp -= 1;
    wave_sync_lds();
    const uint64_t w = c.local[c.lsp];
    wave_sync_lds();
    run_box(c, pi, uniform64((int64_t)w), acc);
  }
}

// The large path for one pair: `task` (a root box, a queued box or a leaf
// tile) goes on the wave's box stack and the stack is drained.  Every large
// box of the kernel goes through this one site.  Returns the intersection
// counted.
__device__ __forceinline__ uint64_t run_large(Ctx& c, const PairInfo& pi, uint64_t task) {
  c.local[c.lsp] = task;
  c.lsp += 1;
  wave_sync_lds();
  uint64_t acc = 0;
  drain_local(c, pi, acc);
  return acc;
}

// The task word of a whole pair box: a cell of the first level whose side
// covers the box, at the pair-box origin.
__device__ __forceinline__ uint64_t root_task(const PairInfo& pi) {
  const int side = max(pi.box.x1 - pi.box.x0, pi.box.y1 - pi.box.y0);
  int cl = 0;
  while ((kTile << (3 * cl)) < side) ++cl;
  return task_word(pi.hidx < 0 ? 0 : pi.hidx, cl, 0, 0, false, false);
}

// A listed pair (its box from the medium sweep).  Its index also
// names it in the task words of its boxes.
__device__ __forceinline__ PairInfo heavy_info(const BatchArgs& a, int64_t pair) {
  PairInfo pi;
  pi.hidx = pair;
  pi.pair = pair;
  const int64_t ia = a.pa[pair], ib = a.pb[pair];
  pi.op = a.A.off[ia];
  pi.np = a.A.off[ia + 1] - pi.op;
  pi.oq = a.B.off[ib];
  pi.nq = a.B.off[ib + 1] - pi.oq;
  pi.box = load_meta(a.hbox, pair);
  pi.area_sum = 0;
  make_uniform(pi);
  return pi;
}

// The list bucket of a pair with n vertices (largest first; one bucket when
// the order is switched off).
__device__ __forceinline__ int lpt_bucket(uint32_t flags, int64_t h, int64_t n) {
  if (flags & SCCG_F_NO_LPT) return 0;
  return n >= 4 * h ? 3 : n >= 2 * h ? 2 : n >= h ? 1 : 0;
}

// Occupancy target of the persistent kernel (waves per SIMD); 0 leaves the
// register budget to the compiler.  A build-time tuning knob.
#ifndef SCCG_RUN_WAVES_PER_EU
#define SCCG_RUN_WAVES_PER_EU 4
#endif
#if SCCG_RUN_WAVES_PER_EU > 0
#define SCCG_RUN_ATTR __attribute__((amdgpu_waves_per_eu(SCCG_RUN_WAVES_PER_EU)))
#else
#define SCCG_RUN_ATTR
#endif

// -------------------------------------------------------------------- sweep
// First pass of a batched call: every pair, one at a time per wave.  A wave
// looks at up to 64 pairs of its share at once, a pair per lane: index check,
// ring offsets and lengths, and the class.  Long pairs (a ring over
// kMediumRing vertices, or heavy_verts in all) and medium ones (a ring over
// kSweepRing vertices, or an empty one) are listed for the second pass.  Of
// the others the wave holds both rings in registers, the next pair's loads in
// flight; when the union of their MBRs fits one leaf tile the pair is counted
// there at once (below Section 3.4's pixelization threshold, I and U
// directly), else it is listed as well, as is a union box of exactly 64 rows
// (see box_count).
constexpr int kUnionChunks = 3;                       // 64-vertex chunks per ring in the union sweep
constexpr int kMediumChunks = 4;                      // and in the medium sweep
constexpr int kSweepRing = kUnionChunks * kWave;      // longest ring of the union sweep
constexpr int kMediumRing = kMediumChunks * kWave;    // longest ring of the medium sweep
constexpr int kSweepWaves = 4;                        // waves per workgroup of the sweep
// Occupancy targets (waves per SIMD) and the tiles of a team's stripes,
// build-time tuning knobs.  The union sweep waits on memory where rings are
// short (200,000 uniform pairs: 101 -> 76 us, 4.1 TB/s of rings; the heavy-tailed
// 2M 570 + 38 of a setup pass -> 494 us): eight waves beat seven by 2 %, and
// with pair boxes (2.6M candidate pairs of dense tiles) 1159 us against 1213
// with seven and 1294 with six.
#ifndef SCCG_TEAM_TILES
#define SCCG_TEAM_TILES 14
#endif
#ifndef SCCG_MEDIUM_WAVES_PER_EU
#define SCCG_MEDIUM_WAVES_PER_EU 5
#endif
#ifndef SCCG_SWEEP_WAVES_PER_EU
#define SCCG_SWEEP_WAVES_PER_EU 8
#endif
#ifndef SCCG_RUN_STEAL
#define SCCG_RUN_STEAL 0
#endif
// whether the persistent kernel's waves also claim listed pairs from other
// XCDs' streams
constexpr bool kRunSteal = SCCG_RUN_STEAL != 0;

// the lanes named by a wave-uniform mask (the mask is the lane condition)
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Lane L < 32 gets lane L + 32's value (v_permlane32_swap).
__device__ __forceinline__ uint32_t upper_half(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_permlane32_swap((int)v, (int)v, false, false)[1];
}
__device__ __forceinline__ uint64_t upper_half(uint64_t v) {
  return ((uint64_t)upper_half((uint32_t)(v >> 32)) << 32) | upper_half((uint32_t)v);
}
// m & the other half's m, in every lane
__device__ __forceinline__ uint32_t both_halves(uint32_t v) {
  const auto s = __builtin_amdgcn_permlane32_swap((int)v, (int)v, false, false);
  return (uint32_t)s[0] & (uint32_t)s[1];
}
__device__ __forceinline__ uint64_t both_halves(uint64_t v) {
  return ((uint64_t)both_halves((uint32_t)(v >> 32)) << 32) | both_halves((uint32_t)v);
}

// A pair in registers: each ring in up to N 64-vertex chunks, lane L of chunk
// c holding vertex 64 c + L.
template <int N>
struct PairRegs {
  int2 p[N], q[N];
};

// Extents of a lane's vertices, minima and complemented maxima, so that all
// four reduce by minimum.
struct Ext {
  int x0, y0, nx1, ny1;
};
__device__ __forceinline__ Ext ext_of(int2 v) { return Ext{v.x, v.y, ~v.x, ~v.y}; }
__device__ __forceinline__ void ext_add(Ext& e, int2 v) {
  e = Ext{min(e.x0, v.x), min(e.y0, v.y), min(e.nx1, ~v.x), min(e.ny1, ~v.y)};
}
// Wave minimum of four values at once: two half swaps and a row swap leave
// each value in one row of 16 lanes, which four row steps reduce together
// (10 steps for the four, where a reduction of each takes 24).
__device__ __forceinline__ Ext wave_min4(const Ext& e) {
  const auto s0 = __builtin_amdgcn_permlane32_swap(e.x0, e.y0, false, false);
  const auto s1 = __builtin_amdgcn_permlane32_swap(e.nx1, e.ny1, false, false);
  const int a = min((int)s0[0], (int)s0[1]), b = min((int)s1[0], (int)s1[1]);
  const auto s2 = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  int x = min((int)s2[0], (int)s2[1]);
  x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0xb1, 0xf, 0xf, false));
  x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x4e, 0xf, 0xf, false));
  x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x141, 0xf, 0xf, false));
  x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x140, 0xf, 0xf, false));
  return Ext{__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 16),
             __builtin_amdgcn_readlane(x, 48)};
}
__device__ __forceinline__ Meta meta_of(const Ext& e) { return Meta{e.x0, e.y0, ~e.nx1, ~e.ny1}; }
__device__ __forceinline__ bool out_of_range(const Meta& m) {
  return m.x0 < -kMaxCoord || m.y0 < -kMaxCoord || m.x1 > kMaxCoord || m.y1 > kMaxCoord;
}

// The share of n items of one wave of a launch whose workgroups have `per_wg`
// waves: runs of at most `longest` consecutive items, interleaved over the
// waves so that all of them work in the same part of the list, with the waves
// in an order that puts neighbouring runs on one XCD (rings that neighbouring
// pairs share stay in its L2).
struct WaveShare {
  uint32_t count;  // items of this wave
  uint32_t me, n_waves, run;
  __device__ __forceinline__ WaveShare(uint32_t n, int per_wg, int w, int longest) {
    const unsigned g = gridDim.x, b = blockIdx.x;
    const unsigned at = g % kStreams == 0 ? (b % kStreams) * (g / kStreams) + b / kStreams : b;
    n_waves = uniform_u(g * (unsigned)per_wg);
    me = uniform_u(at * (unsigned)per_wg + (unsigned)w);
    run = uniform_u(max(1u, min((uint32_t)longest, n / (n_waves * 32u))));  // as share_run
    const uint32_t round = n_waves * run, full = n / round, rest = n - full * round, before = me * run;
    count = uniform_u(full * run + (rest > before ? min(run, rest - before) : 0u));
  }
  // the list index of the wave's item k
  __device__ __forceinline__ uint32_t entry(uint32_t k) const {
    const uint32_t turn = run == 1u ? k : k / run;
    return (turn * n_waves + me) * run + (k - turn * run);
  }
};

// A list that the workgroups of every stream appended a part of their own to,
// taken as one: the parts' lengths, and where its entry e stands.
struct ListParts {
  uint32_t n[kStreams], total;
  __device__ __forceinline__ void read(const Counter* count) {
    total = 0;
#pragma unroll
    for (int st = 0; st < kStreams; ++st) {
      n[st] = uniform_u((uint32_t)count[st].v);
      total += n[st];
    }
  }
  // the lengths in the lanes from `lane` on
  __device__ __forceinline__ void of_lanes(int length, int lane) {
    total = 0;
#pragma unroll
    for (int st = 0; st < kStreams; ++st) {
      n[st] = (uint32_t)__builtin_amdgcn_readlane(length, lane + st);
      total += n[st];
    }
  }
  __device__ __forceinline__ int64_t at(uint32_t e, int64_t stream_cap) const {
    int64_t part = 0;
    bool found = false;
#pragma unroll
    for (int st = 0; st < kStreams; ++st) {
      found = found || e < n[st];
      if (!found) {
        e -= n[st];
        part += stream_cap;
      }
    }
    return part + e;
  }
};

// The lists of all buckets and streams, taken as one, the largest bucket first:
// lane L < kParts has that of stream L % kStreams of bucket kLptBuckets - 1 -
// L / kStreams.
constexpr int kParts = kLptBuckets * kStreams;
struct BucketLists {
  int first;    // where the lane's list begins in the whole
  int64_t all;  // entries of all
  __device__ __forceinline__ static int bucket(int part) { return kLptBuckets - 1 - part / kStreams; }
  // length: of the lane's list (0 in the lanes from kParts on)
  __device__ __forceinline__ BucketLists(int length, int lane) {
    first = length;
#pragma unroll
    for (int d = 1; d < kParts; d <<= 1) {
      const int v = __shfl_up(first, d, kWave);
      if (lane >= d) first += v;
    }
    all = __builtin_amdgcn_readlane(first, kParts - 1);
    first -= length;
  }
  // where entry k stands in lists of `cap` entries each
  __device__ __forceinline__ int64_t at(int64_t k, int64_t cap, int lane) const {
    const int part = kWave - 1 - __clzll((long long)ballot(lane < kParts && first <= (int)k));
    return (int64_t)(bucket(part) * kStreams + part % kStreams) * cap + (k - __builtin_amdgcn_readlane(first, part));
  }
};

// Both rings of a pair, as the pair arrays and the offsets give them.
struct PairRec {
  int64_t op, oq;
  int32_t np, nq;
};
__device__ __forceinline__ PairRec pair_rec(const BatchArgs& a, int64_t ia, int64_t ib) {
  PairRec r;
  r.op = a.A.off[ia];
  r.oq = a.B.off[ib];
  r.np = (int32_t)(a.A.off[ia + 1] - r.op);
  r.nq = (int32_t)(a.B.off[ib + 1] - r.oq);
  return r;
}
// Lane j's record, in every lane.
__device__ __forceinline__ PairRec rec_of_lane(const PairRec& r, int j) {
  return PairRec{readlane64(r.op, j), readlane64(r.oq, j), __builtin_amdgcn_readlane(r.np, j),
                 __builtin_amdgcn_readlane(r.nq, j)};
}

// Append each lane's value to a list, for the lanes in `m`, with one
// reservation.
__device__ __forceinline__ void list_append(unsigned long long& count, int32_t* list, uint64_t m, int32_t value, int lane) {
  unsigned long long base = 0;
  if (lane == 0) base = atomicAdd(&count, (unsigned long long)__popcll(m));
  base = (unsigned long long)uniform64((int64_t)__shfl((long long)base, 0, kWave));
  if (lane_in(m)) list[base + (unsigned long long)lanes_below(m)] = value;
}

// Claim a chunk of `chunk` consecutive entries from per-stream counters (one
// stream per XCD, exhausted streams marked in `empty`): its first entry, or
// -1 when every stream is exhausted.
__device__ __forceinline__ int64_t claim_chunk(Counter* next, int64_t n, int chunk, int xcd, int lane,
                                               uint32_t& empty) {
  const unsigned long long n_chunks = ((unsigned long long)n + chunk - 1) / chunk;
  if (n_chunks == 0) empty = 0xffu;
  while (empty != 0xffu) {
    const int st = next_stream(empty, xcd);
    unsigned long long k = 0;
    if (lane == 0) k = atomicAdd(&next[st].v, 1ull);
    k = (unsigned long long)uniform64((int64_t)__shfl((long long)k, 0, kWave));
    const unsigned long long g = k * kStreams + st;
    if (g >= n_chunks) {
      empty = uniform_u(empty | (1u << st));
      continue;
    }
    return uniform64((int64_t)g * chunk);
  }
  return -1;
}

// The batched state needs no reset of its own before a call: each kernel
// leaves what it is done with ready for the next one, in the order of the
// stream.
//   - The sweep (this function, all workgroups) clears the queue slots the
//     previous call used and, in its first workgroup, the counters that only
//     the later kernels of a call touch.
//   - The medium sweep sets the queues' heads and tails back (the sweep has
//     just used them to find those slots).
//   - The persistent kernel sets the counts of the lists that the sweep
//     appends to back (the medium sweep has read them).
__device__ __forceinline__ void next_call_state(const BatchArgs& a) {
  BatchState& st = *a.st;
  const unsigned t = threadIdx.x;
  if (blockIdx.x == 0) {
    if (t < (unsigned)kStreams) {
      st.p_next[t].v = 0;
      st.l_next[t].v = 0;
    }
    if (t < (unsigned)(kLptBuckets * kStreams)) st.l_count[t % kStreams].v[t / kStreams] = 0;
  }
  // most calls used none: every counter in one load (one after the other, eight
  // latencies were half of a small call's sweep)
  const int lane = lane_id();
  unsigned long long mine = 0;
  if (lane < a.n_queues) mine = max(st.q_tail[lane].v, st.q_head[lane].v);
  for (uint64_t some = ballot(mine != 0); some; some &= some - 1) {
    const int q = __ffsll((long long)some) - 1;
    unsigned long long used = (unsigned long long)readlane64((int64_t)mine, q);
    if (used > (unsigned long long)a.queue_cap) used = (unsigned long long)a.queue_cap;
    unsigned long long* base = a.queue + (size_t)q * a.queue_cap;
    for (unsigned long long k = (unsigned long long)blockIdx.x * blockDim.x + t; k < used;
         k += (unsigned long long)gridDim.x * blockDim.x)
      base[k] = 0;
  }
}

// --------------------------------------------------- rings of the union sweep
// Pixel (x, y) is inside a ring iff an odd number of its vertical edges lie
// right of x with a span holding row y (Section 3.1).  A vertical edge from
// (X, ya) to (X, yb) holds row y iff exactly one of ya, yb is <= y, so its
// term is the XOR of one term per end: "rows >= y_end, in the columns left of
// X".  Summed over a ring, a vertex contributes its term once for each
// vertical edge it bounds: once at a corner, twice (no effect) between two
// vertical edges, never between two horizontal ones.  So every vertex whose
// two edges are not both vertical or both horizontal XORs the mask of rows
// >= y_v into the slot of the rightmost column left of x_v, and the prefix
// XOR over the columns (lanes, in reverse order as in the other leaves)
// gives every column's crossing parities (the vertex form of the test).

// Where the slots of one wave stand.  Column k from the right of a ring has
// slot k; slot W takes the corners on the tile's left side, which have no
// column left of them, and is never read.
//   halves (W = 32): p's slots are 0-32, q's from 34, so that lane L < 32
//     reads p's slot L and the others q's slot L - 32 at L + 2;
//   else (W = 64): p's are 0-64, q's from 66.
constexpr int kHalfQ = 34, kFullQ = 66;
constexpr int kSweepSlots = 132;
// kPairBox: after them q's tile, with a tile of nothing on both sides of it
constexpr int kTileQ = kSweepSlots + kWave;
constexpr int kPairBoxSlots = kSweepSlots + 3 * kWave;

// The lanes whose vertex has a vertical edge to its successor, in a chunk
// whose lanes past the ring's end hold the first vertex again: the next lane,
// and for lane 63 lane 0 of `after` (the last lane of its rotation) or of the
// chunk itself.
__device__ __forceinline__ uint64_t vertical_edges(int x, int after) {
  const int t = __builtin_amdgcn_update_dpp(0, after, 0x134, 0xf, 0xf, false);  // wave_rol:1
  return ballot(x == __builtin_amdgcn_update_dpp(t, x, 0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ uint64_t vertical_edges(int x) {
  return ballot(x == __builtin_amdgcn_update_dpp(0, x, 0x134, 0xf, 0xf, false));
}

// XOR a chunk's corners (the lanes `corners`) into the slots at `base`, of a
// tile of W columns and R rows whose right side is at x1 and bottom at y0.
// kClip: vertices may lie outside the tile (see box_count).
template <int W, typename M, bool kClip>
__device__ __forceinline__ void chunk_xor(M* base, int2 v, uint64_t corners, int x1, int y0) {
  constexpr int R = (int)sizeof(M) * 8;
  if (kClip) {
    v.x = clamp_to(v.x, x1 - W, x1);
    v.y = clamp_to(v.y, y0, y0 + R - 1);
  }
  const int pos = x1 - v.x, ty = v.y - y0;
  if (lane_in(corners)) slot_xor(base + pos, 0, (M)(~(M)0 << ty));
}

// The corners of a whole ring into its slots (kOne: of at most 64 vertices).
// The chunks come by value: by reference the compiler merges the calls below
// on a chosen address, and the registers become memory.
template <int W, typename M, bool kClip, bool kOne>
__device__ __forceinline__ void ring_xor(M* base, int2 d0, int2 d1, int2 d2, int nr, int x1, int y0) {
  static_assert(kUnionChunks == 3, "the chunks of a sweep ring");
  if (kOne || nr <= kWave) {
    const uint64_t b = vertical_edges(d0.x);
    const uint64_t corners = (b ^ ((b << 1) | ((b >> (nr - 1)) & 1ull))) & (~0ull >> (kWave - nr));
    chunk_xor<W, M, kClip>(base, d0, corners, x1, y0);
  } else if (nr <= 2 * kWave) {
    const uint64_t b0 = vertical_edges(d0.x, d1.x), b1 = vertical_edges(d1.x, d0.x);
    const uint64_t in = ~0ull >> (2 * kWave - nr);
    chunk_xor<W, M, kClip>(base, d0, b0 ^ ((b0 << 1) | ((b1 >> (nr - 1 - kWave)) & 1ull)), x1, y0);
    chunk_xor<W, M, kClip>(base, d1, (b1 ^ ((b1 << 1) | (b0 >> 63))) & in, x1, y0);
  } else {
    const uint64_t b0 = vertical_edges(d0.x, d1.x), b1 = vertical_edges(d1.x, d2.x), b2 = vertical_edges(d2.x, d0.x);
    const uint64_t in = ~0ull >> (3 * kWave - nr);
    chunk_xor<W, M, kClip>(base, d0, b0 ^ ((b0 << 1) | ((b2 >> (nr - 1 - 2 * kWave)) & 1ull)), x1, y0);
    chunk_xor<W, M, kClip>(base, d1, b1 ^ ((b1 << 1) | (b0 >> 63)), x1, y0);
    chunk_xor<W, M, kClip>(base, d2, (b2 ^ ((b2 << 1) | (b1 >> 63))) & in, x1, y0);
  }
}

// Counts of a pair on the tile at (x0, y0), W = 32 or 64 columns wide, M's
// bits tall: twice I in the high half of the word, |p| + |q| within the tile
// in the low half, summed over the wave.  Rows and columns of the tile past
// the union box come out outside.
template <bool kHalves, typename M, bool kClip, bool kOne>
__device__ __forceinline__ uint32_t tile_counts(uint64_t* words, int lane, const PairRegs<kUnionChunks>& r, int np,
                                                int nq, int x0, int y0) {
  constexpr int W = kHalves ? 32 : kWave;
  M* slots = reinterpret_cast<M*>(words);
  M* mine = slots + (kHalves ? lane + 2 * (lane >> 5) : lane);
  *mine = (M)0;
  if (!kHalves) mine[kFullQ] = (M)0;
  wave_sync_lds();
  ring_xor<W, M, kClip, kOne>(slots, r.p[0], r.p[1], r.p[2], np, x0 + W, y0);
  ring_xor<W, M, kClip, kOne>(slots + (kHalves ? kHalfQ : kFullQ), r.q[0], r.q[1], r.q[2], nq, x0 + W, y0);
  wave_sync_lds();
  uint32_t t;
  if (kHalves) {
    const M m = wave_prefix_xor<true>(*mine);
    // both halves hold the columns' common pixels
    t = (uint32_t)__popcll((uint64_t)m) + ((uint32_t)__popcll((uint64_t)both_halves(m)) << 16);
  } else {
    const M mp = wave_prefix_xor<false>(*mine);
    const M mq = wave_prefix_xor<false>(mine[kFullQ]);
    t = (uint32_t)__popcll((uint64_t)mp) + (uint32_t)__popcll((uint64_t)mq) +
        ((uint32_t)__popcll((uint64_t)(mp & mq)) << 17);
  }
  wave_sync_lds();
  return wave_sum_u32(t);
}

// The counts of a pair on a box at most 64 wide and less than 64 tall (see
// tile_counts): the union of its MBRs, or, kClip, its pair box.  There a
// corner left of the box toggles none of its columns and one right of it all
// of them; one below it counts as standing in its first row, and one above
// the tile's last row in that row, where every column then has as many
// corners as the ring has right of it, an even number: outside, as a row
// above the box has to be for the intersection.  (A box of 64 rows has no
// such row in the tile: the medium sweep takes it.)
template <bool kClip, bool kOne>
__device__ __forceinline__ uint32_t box_count(uint64_t* words, int lane, const PairRegs<kUnionChunks>& r, int np, int nq,
                                              int x0, int y0, uint32_t w, uint32_t h) {
  if (w <= 32u)
    return h < 32u ? tile_counts<true, uint32_t, kClip, kOne>(words, lane, r, np, nq, x0, y0)
                   : tile_counts<true, uint64_t, kClip, kOne>(words, lane, r, np, nq, x0, y0);
  return h < 32u ? tile_counts<false, uint32_t, kClip, kOne>(words, lane, r, np, nq, x0, y0)
                 : tile_counts<false, uint64_t, kClip, kOne>(words, lane, r, np, nq, x0, y0);
}
template <bool kClip>
__device__ __forceinline__ uint32_t box_count(uint64_t* words, int lane, const PairRegs<kUnionChunks>& r, int np, int nq,
                                              bool one, int x0, int y0, uint32_t w, uint32_t h) {
  return one ? box_count<kClip, true>(words, lane, r, np, nq, x0, y0, w, h)
             : box_count<kClip, false>(words, lane, r, np, nq, x0, y0, w, h);
}

// The parities of a ring on its own tile at (x0, y0), 64 x 64, which it does
// not fill to the top row: lane L has column x0 + 63 - L.
template <bool kOne>
__device__ __forceinline__ uint64_t ring_tile(uint64_t* slots, int lane, int2 d0, int2 d1, int2 d2, int nr, int x0,
                                              int y0) {
  slots[lane] = 0;
  wave_sync_lds();
  ring_xor<kWave, uint64_t, false, kOne>(slots, d0, d1, d2, nr, x0 + kWave, y0);
  wave_sync_lds();
  const uint64_t m = wave_prefix_xor<false>(slots[lane]);
  wave_sync_lds();
  return m;
}
__device__ __forceinline__ uint64_t ring_tile(uint64_t* slots, int lane, const int2 (&d)[kUnionChunks], int nr, int x0,
                                              int y0) {
  return nr <= kWave ? ring_tile<true>(slots, lane, d[0], d[1], d[2], nr, x0, y0)
                     : ring_tile<false>(slots, lane, d[0], d[1], d[2], nr, x0, y0);
}
// whether a ring's tile holds it (see ring_tile)
__device__ __forceinline__ bool on_one_tile(const Meta& m) {
  return !out_of_range(m) && max(side_u(m.x0, m.x1), side_u(m.y0, m.y1) + 1u) <= (uint32_t)kTile;
}
// pixels of a mask over the wave
__device__ __forceinline__ uint32_t wave_pixels(uint64_t m) { return wave_sum_u32((uint32_t)__popcll(m)); }

// Twice the signed area of a ring at most kMaxSide wide and tall, summed as
// (x + x') (y' - y) over its edges with x relative to its first vertex,
// modulo 2^32, in which it is exact.
__device__ __forceinline__ int64_t ring_area(const int2 (&d)[kUnionChunks], int nr) {
  const uint32_t f2 = 2u * (uint32_t)__builtin_amdgcn_readlane(d[0].x, 0);
  uint32_t tn = 0;
#pragma unroll
  for (int c = 0; c < kUnionChunks; ++c) {
    if (c * kWave < nr) {
      const int2 f = d[0], g = d[c + 1 < kUnionChunks ? c + 1 : 0];
      const bool more = (c + 1) * kWave < nr;
      const int ax = more ? g.x : f.x, ay = more ? g.y : f.y;
      const int tx = __builtin_amdgcn_update_dpp(0, ax, 0x134, 0xf, 0xf, false);
      const int ty = __builtin_amdgcn_update_dpp(0, ay, 0x134, 0xf, 0xf, false);
      const int sx = __builtin_amdgcn_update_dpp(tx, d[c].x, 0x130, 0xf, 0xf, false);
      const int sy = __builtin_amdgcn_update_dpp(ty, d[c].y, 0x130, 0xf, 0xf, false);
      tn += (uint32_t)__mul24((int)((uint32_t)d[c].x + (uint32_t)sx - f2), (int)((uint32_t)sy - (uint32_t)d[c].y));
    }
  }
  const int32_t t = (int32_t)wave_sum_u32(tn);
  return (t < 0 ? -(int64_t)t : (int64_t)t) / 2;
}

// Vertex 64 c + L of a ring of nr vertices in lane L, the first vertex again
// past its end: neutral for extents, and the last vertex's successor comes
// out right.  Only the chunks the ring has are loaded.
typedef const char __attribute__((address_space(1))) * ring_ptr;
__device__ __forceinline__ void ring_load(ring_ptr ring, int nr, int lane, int2 (&d)[kUnionChunks]) {
#pragma unroll
  for (int c = 0; c < kUnionChunks; ++c) {
    if (c == 0 || c * kWave < nr) {
      const uint32_t at = c * kWave + lane < nr ? (uint32_t)(c * kWave + lane) * 8u : 0u;
      const uint64_t v = *reinterpret_cast<const uint64_t __attribute__((address_space(1)))*>(ring + at);
      d[c] = make_int2((int)(uint32_t)v, (int)(uint32_t)(v >> 32));
    }
  }
}
__device__ __forceinline__ void ring_move(int2 (&to)[kUnionChunks], const int2 (&from)[kUnionChunks], int nr) {
  to[0] = from[0];
#pragma unroll
  for (int c = 1; c < kUnionChunks; ++c)
    if (c * kWave < nr) to[c] = from[c];
}
// extents of a ring's lanes
__device__ __forceinline__ Ext ring_ext(int2 d0, int2 d1, int2 d2, int nr) {
  Ext e = ext_of(d0);
  if (nr > kWave) ext_add(e, d1);
  if (nr > 2 * kWave) ext_add(e, d2);
  return e;
}

// The lanes' records of up to 64 sweep pairs: both rings' addresses and
// lengths (np | nq << 16; each 1 to kSweepRing).
struct SweepRecs {
  uint64_t p, q;
  uint32_t n;
};
// one of them, wave-uniform
struct SweepPair {
  ring_ptr p, q;
  int np, nq;
};
__device__ __forceinline__ SweepPair sweep_pair(const SweepRecs& r, int j) {
  const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)r.n, j);
  return SweepPair{(ring_ptr)readlane64((int64_t)r.p, j), (ring_ptr)readlane64((int64_t)r.q, j), (int)(n & 0xffffu),
                   (int)(n >> 16)};
}

// ------------------------------------------------------------- rings' tiles
// The tiles of all rings of both sets, for a call with more pairs than rings
// (use_ring_tiles): a ring per wave, the next one's loads in flight.  1.22M
// rings of 96 vertices: 337 us, 930 MB of rings read and some 350 MB of tiles
// written (3.8 TB/s).
template <bool kStats>
__global__ void __launch_bounds__(kSweepWaves* kWave)
    __attribute__((amdgpu_waves_per_eu(SCCG_SWEEP_WAVES_PER_EU)))
k_ring_tiles(BatchArgs args) {
  constexpr int kSlots = kWave + 2;
  __shared__ __align__(16) uint64_t tile_slots[kSweepWaves * kSlots];
  Ctx c;
  c.a = &args;
  c.stats = kStats;
  c.lane = lane_id();
  c.slots = tile_slots + (threadIdx.x / kWave) * kSlots;
  const BatchArgs& a = args;
  const int lane = c.lane;
  if (blockIdx.x == 0 && threadIdx.x < (unsigned)kStreams) a.st->t_count[threadIdx.x].v = 0;
  const uint32_t n_a = (uint32_t)a.A.n;
  const int64_t end_a = a.A.n > 0 ? a.A.off[a.A.n] : 0, end_b = a.B.n > 0 ? a.B.off[a.B.n] : 0;
  const WaveShare share(n_a + (uint32_t)a.B.n, kSweepWaves, uniform((int)(threadIdx.x / kWave)), a.chunk);
#pragma unroll 1
  for (uint32_t k0 = 0; k0 < share.count; k0 += kWave) {
    const int cnt = uniform((int)min((uint32_t)kWave, share.count - k0));
    const uint32_t r = share.entry(k0 + (uint32_t)lane);  // the lane's ring
    uint64_t at = 0;
    uint32_t nv = 0;
    if (lane < cnt) {
      const bool of_b = r >= n_a;
      const int64_t* off = of_b ? a.B.off + (r - n_a) : a.A.off + r;
      const int64_t o = off[0], n = off[1] - o;
      at = (uint64_t)((of_b ? a.B.xy : a.A.xy) + o);
      // a ring that no pair names may have any offsets: read within the vertices only
      const bool within = o >= 0 && off[1] <= (of_b ? end_b : end_a);
      nv = within && n >= 1 && n <= kSweepRing ? (uint32_t)n : 0u;
    }
    Meta box{0, 0, 0, 0};  // the lane's ring's
    uint2 sums = make_uint2(0, 0);
    uint64_t todo = ballot(nv > 0);
    int2 cur[kUnionChunks], nxt[kUnionChunks];
    int j = 0, n = 0;
    if (todo) {
      j = __ffsll((long long)todo) - 1;
      n = __builtin_amdgcn_readlane((int)nv, j);
      ring_load((ring_ptr)readlane64((int64_t)at, j), n, lane, cur);
    }
#pragma unroll 1
    while (todo) {
      todo &= todo - 1;
      const Meta m = meta_of(wave_min4(ring_ext(cur[0], cur[1], cur[2], n)));
      int jn = j, nn = n;
      if (todo) {
        jn = __ffsll((long long)todo) - 1;
        nn = __builtin_amdgcn_readlane((int)nv, jn);
        ring_load((ring_ptr)readlane64((int64_t)at, jn), nn, lane, nxt);
      }
      if (on_one_tile(m)) {
        const uint64_t t = ring_tile(c.slots, lane, cur, n, m.x0, m.y0);
        const uint32_t ring = (uint32_t)__builtin_amdgcn_readlane((int)r, j);
        const int col = kWave - 1 - lane;
        if (col < m.x1 - m.x0) a.ring_tiles[(uint64_t)ring * kTile + col] = t;
        const uint32_t held = wave_pixels(t) | (uint32_t)n << 16, area = (uint32_t)ring_area(cur, n);
        const bool me = lane == j;
        box = Meta{me ? m.x0 : box.x0, me ? m.y0 : box.y0, me ? m.x1 : box.x1, me ? m.y1 : box.y1};
        sums = make_uint2(me ? held : sums.x, me ? area : sums.y);
        if (kStats) stat_add(c, 14, (unsigned long long)n);
      }
      j = jn;
      n = nn;
      ring_move(cur, nxt, n);
    }
    if (lane < cnt) {
      *reinterpret_cast<int4*>(a.ring_box + r) = make_int4(box.x0, box.y0, box.x1, box.y1);
      a.ring_sums[r] = sums;
    }
  }
}

// A pair of rings with tiles: their pair box in both tiles.
struct TilePair {
  uint32_t at_p, at_q;  // bytes from ring_tiles to the box's first column
  uint32_t how;         // columns, then the shifts that bring p's and q's rows together (8 bits each)
  uint32_t n;           // pixels in common
};

// The pixels in common of 64 pairs (of no columns: none), into their entries:
// 16 lanes per pair, two columns per lane and step, eight pairs' columns in
// flight while the eight before are counted.  Lanes past the box read its
// first columns.
__device__ __forceinline__ void count_tile_pairs(const BatchArgs& a, TilePair* pairs, int lane) {
  typedef uint64_t cols2 __attribute__((ext_vector_type(2), aligned(8)));
  typedef const char __attribute__((address_space(1))) * tile_ptr;
  typedef const cols2 __attribute__((address_space(1))) * cols_ptr;
  const tile_ptr tiles = (tile_ptr)(uint64_t)a.ring_tiles;
  const uint32_t first = 2u * ((uint32_t)lane & 15u);
  struct Step {
    uint32_t how[2];
    cols2 p[2], q[2];
  };
  auto load = [&](Step& d, int t, uint32_t col) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const TilePair x = pairs[4 * (t + u) + (lane >> 4)];
      const uint32_t o = col < (x.how & 0xffu) ? col * 8u : 0u;
      d.how[u] = x.how;
      d.p[u] = *(cols_ptr)(tiles + (x.at_p + o));
      d.q[u] = *(cols_ptr)(tiles + (x.at_q + o));
    }
  };
  auto count = [&](const Step& d, uint32_t col, uint32_t (&n)[2]) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t w = d.how[u] & 0xffu, sp = (d.how[u] >> 8) & 0xffu, sq = d.how[u] >> 16;
      const uint64_t m0 = (d.p[u].x << sp) & (d.q[u].x << sq), m1 = (d.p[u].y << sp) & (d.q[u].y << sq);
      n[u] += (col < w ? (uint32_t)__popcll(m0) : 0u) + (col + 1u < w ? (uint32_t)__popcll(m1) : 0u);
    }
  };
  Step cur, nxt;
  load(cur, 0, first);
#pragma unroll 1
  for (int t = 0; t < kWave / 4; t += 2) {
    load(nxt, min(t + 2, kWave / 4 - 2), first);
    uint32_t n[2] = {0, 0};
    count(cur, first, n);
    if (ballot(max(cur.how[0] & 0xffu, cur.how[1] & 0xffu) > 32u)) {
      load(cur, t, first + 32u);
      count(cur, first + 32u, n);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t v = n[u];
      v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, false);
      v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, false);
      v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false);
      v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, false);
      if (first == 0) pairs[4 * (t + u) + (lane >> 4)].n = v;
    }
    cur = nxt;
  }
}

// The pairs whose rings both have a tile and that are no long pairs: their
// counts, a pair per lane up to its box, then count_tile_pairs.  2.69M pairs:
// 210 us, waiting on the tiles (0.7 GB from HBM, 2 GB through the L2s); with
// the loads of a step waited for at once it was 337.  The others are listed for the union sweep (where the persistent kernel's lists will be,
// which is not written before it).  One register less than eight waves leave:
// 64-bit shifts by a count in the last register of the allocation came out
// with another count in some lanes.
template <bool kStats>
__global__ void __launch_bounds__(kSweepWaves* kWave)
    __attribute__((amdgpu_waves_per_eu(SCCG_SWEEP_WAVES_PER_EU), amdgpu_num_vgpr(31)))
k_tile_pairs(BatchArgs args) {
  __shared__ TilePair pair_slots[kSweepWaves * kWave];
  const BatchArgs& a = args;
  const int lane = lane_id(), w = uniform((int)(threadIdx.x / kWave));
  TilePair* pairs = pair_slots + w * kWave;
  const bool direct = direct_union(a), union_ok = direct || !(a.flags & SCCG_F_NO_UNION_TILE);
  const WaveShare share((uint32_t)a.n_pairs, kSweepWaves, w, a.chunk);
#pragma unroll 1
  for (uint32_t k0 = 0; k0 < share.count; k0 += kWave) {
    const uint32_t i = share.entry(k0 + (uint32_t)lane);
    const bool some = lane < (int)min((uint32_t)kWave, share.count - k0);
    bool quick = false;
    uint32_t areas = 0;
    TilePair mine{0, 0, 0, 0};
    int32_t ia = -1, ib = -1;
    if (some) {
      ia = a.pa[i];
      ib = a.pb[i];
    }
    if (ia >= 0 && ia < a.A.n && ib >= 0 && ib < a.B.n) {
      const uint32_t rq = (uint32_t)a.A.n + (uint32_t)ib;
      const Meta bp = load_meta(a.ring_box, ia), bq = load_meta(a.ring_box, rq);
      const uint2 sp = a.ring_sums[ia], sq = a.ring_sums[rq];
      const uint32_t np = sp.x >> 16, nq = sq.x >> 16;
      const Meta un = union_box(bp, bq), box = pair_box(bp, bq);
      const bool on_union = union_ok && max(side_u(un.x0, un.x1), side_u(un.y0, un.y1)) <= (uint32_t)kTile;
      quick = np && nq && (int)(np + nq) < a.heavy_verts && (on_union || !direct);
      areas = on_union ? (sp.x & 0xffffu) + (sq.x & 0xffffu) : sp.y + sq.y;
      if (quick && box.x0 < box.x1 && box.y0 < box.y1) {
        const int dy = bp.y0 - bq.y0;  // less than a tile's side, as the boxes meet
        mine.at_p = ((uint32_t)ia * kTile + (uint32_t)(box.x0 - bp.x0)) * 8u;
        mine.at_q = (rq * kTile + (uint32_t)(box.x0 - bq.x0)) * 8u;
        mine.how = (uint32_t)(box.x1 - box.x0) | (uint32_t)max(dy, 0) << 8 | (uint32_t)max(-dy, 0) << 16;
      }
      if (kStats && quick) {
        const Meta over = on_union ? un : box;
        const bool none = over.x0 >= over.x1 || over.y0 >= over.y1;
        const unsigned long long nv = np + nq,
                                 px = none ? 0ull : (unsigned long long)side_u(over.x0, over.x1) * side_u(over.y0, over.y1);
        unsigned long long* st = a.st->stats;
        atomicAdd(st + (on_union ? 13 : 12), nv);
        atomicAdd(st + (none ? 7 : 5), 1ull);
        atomicAdd(st + 11, px);
        atomicAdd(st + 1, 1ull);
        atomicAdd(st + 0, 2ull * px);
        atomicAdd(st + 10, nv);
      }
    }
    const uint64_t left = ballot(some && !quick);
    const int st = (int)(blockIdx.x % (unsigned)kStreams);
    if (left) list_append(a.st->t_count[st].v, a.run_list + st * a.stream_cap, left, (int32_t)i, lane);
    pairs[lane] = mine;
    wave_sync_lds();
    if (ballot(mine.how != 0)) count_tile_pairs(a, pairs, lane);
    wave_sync_lds();
    if (quick) {
      const uint32_t n = pairs[lane].n;
      a.inter[i] = (int64_t)n;
      a.uni[i] = (int64_t)(int32_t)(areas - n);  // signed: see k_batch_sweep
    }
    wave_sync_lds();
  }
}

// kPairBox: pairs whose union box exceeds a leaf tile are counted here as well
// (the same counts as the medium sweep's, without loading the rings again), U
// from the areas.  Each ring is pixelized on a tile of its own, and I counts
// the AND of p's tile and q's, shifted by the distance of their corners; q's
// ring, tile and area are kept while consecutive pairs of the wave share it (a
// join's output grouped by one side repeats it).  A ring that no tile holds
// takes the pair to the pair box, if that fits a tile (both rings scattered,
// the corners right of the box all into one slot: 2.69M candidate pairs of
// dense tiles that were all counted so took 1150 us, from own tiles 1015).
// With ring_tiles this is left with the pairs that they do not hold (100,000 of
// those, 50 us).  A separate instance keeps the
// extra registers off the plain sweep, which most mixes run.  kStats: the
// work counters are kept (an instance of its own, so that the others carry no
// test for them).
template <bool kPairBox, bool kStats>
__global__ void __launch_bounds__(kSweepWaves* kWave)
    __attribute__((amdgpu_waves_per_eu(SCCG_SWEEP_WAVES_PER_EU)))
k_batch_sweep(BatchArgs args) {
  constexpr int kSlots = kPairBox ? kPairBoxSlots : kSweepSlots;
  __shared__ __align__(16) uint64_t sweep_slots[kSweepWaves * kSlots];
  Ctx c;
  c.a = &args;
  c.stats = kStats;
  c.lane = lane_id();
  c.slots = sweep_slots + (threadIdx.x / kWave) * kSlots;
  c.local = nullptr;
  c.lsp = 0;
  c.home = 0;
  c.xcd = 0;
  const BatchArgs& a = args;
  const int lane = c.lane;
  const bool direct = direct_union(a);
  const bool union_ok = direct || !(a.flags & SCCG_F_NO_UNION_TILE);
  const unsigned long long t_start = wave_stamp(a);
  next_call_state(a);
  if (kPairBox) {
    c.slots[kTileQ - kWave + lane] = 0;
    c.slots[kTileQ + kWave + lane] = 0;
  }
  // the pairs: all, or those that the rings' tiles left (single ones: they come
  // in runs, and a share of several runs would take far longer than the others)
  const bool tiled = kPairBox && a.ring_tiles != nullptr;
  ListParts parts;
  if (tiled) parts.read(a.st->t_count);
  const WaveShare share(tiled ? parts.total : (uint32_t)a.n_pairs, kSweepWaves, uniform((int)(threadIdx.x / kWave)),
                        tiled ? 1 : a.chunk);
#pragma unroll 1
  for (uint32_t k0 = 0; k0 < share.count; k0 += kWave) {
    const int cnt = uniform((int)min((uint32_t)kWave, share.count - k0));
    int64_t i = share.entry(k0 + (uint32_t)lane);  // the lane's pair
    if (tiled && lane < cnt) i = a.run_list[parts.at((uint32_t)i, a.stream_cap)];
    SweepRecs rec{0, 0, 0};
    int64_t verts = 0;
    int bucket = -1;  // of a long pair
    bool done = false, medium = false, sweep = false;
    uint32_t out_i = 0, out_u = 0;  // the lane's pair's counts (not kPairBox: both in out_i, see tile_counts)
    if (lane < cnt) {
      const int64_t ia = a.pa[i], ib = a.pb[i];
      if (ia < 0 || ia >= a.A.n || ib < 0 || ib >= a.B.n) {
        latch_error(a.err, kErrIndex);
        done = true;
        if (kStats) atomicAdd(&a.st->stats[7], 1ull);
      } else {
        const PairRec r = pair_rec(a, ia, ib);
        verts = (int64_t)r.np + r.nq;
        if (r.np > kMediumRing || r.nq > kMediumRing || verts >= a.heavy_verts)
          bucket = lpt_bucket(a.flags, a.heavy_verts, verts);
        else if (r.np > kSweepRing || r.nq > kSweepRing || r.np <= 0 || r.nq <= 0 || (!union_ok && !kPairBox))
          medium = true;
        else
          sweep = true;
        rec.p = (uint64_t)(a.A.xy + r.op);
        rec.q = (uint64_t)(a.B.xy + r.oq);
        rec.n = (uint32_t)r.np | (uint32_t)r.nq << 16;
      }
    }
    uint64_t todo = ballot(sweep), finished = ballot(done);
    PairRegs<kUnionChunks> cur, nxt;
    SweepPair s{nullptr, nullptr, 0, 0};
    int j = 0;
    if (todo) {
      j = __ffsll((long long)todo) - 1;
      s = sweep_pair(rec, j);
      ring_load(s.p, s.np, lane, cur.p);
      ring_load(s.q, s.nq, lane, cur.q);
    }
    // kPairBox: the last q ring whose extent (and area, once needed) is held
    ring_ptr q_held = nullptr;
    int q_n = 0;
    Meta mq{0, 0, 0, 0};
    int64_t area_q = -1;
    bool tile_q = false;    // q's tile is in LDS
    uint32_t pixels_q = 0;  // and holds this many
#pragma unroll 1
    while (todo) {
      todo &= todo - 1;
      const bool one = max(s.np, s.nq) <= kWave;
      Meta u;
      Meta mp{0, 0, 0, 0};
      if (kPairBox) {
        mp = meta_of(wave_min4(ring_ext(cur.p[0], cur.p[1], cur.p[2], s.np)));
        if (s.q != q_held || s.nq != q_n) {
          mq = meta_of(wave_min4(ring_ext(cur.q[0], cur.q[1], cur.q[2], s.nq)));
          area_q = -1;
          q_held = s.q;
          q_n = s.nq;
          tile_q = on_one_tile(mq);
          if (tile_q) {
            const uint64_t m = ring_tile(c.slots, lane, cur.q, s.nq, mq.x0, mq.y0);
            c.slots[kTileQ + lane] = m;
            wave_sync_lds();
            pixels_q = wave_pixels(m);
            if (kStats) stat_add(c, 14, (unsigned long long)s.nq);
          }
        }
        u = union_box(mp, mq);
      } else {
        Ext e = ext_of(cur.p[0]);
        ext_add(e, cur.q[0]);
        if (!one) {
          if (s.np > kWave) ext_add(e, cur.p[1]);
          if (s.nq > kWave) ext_add(e, cur.q[1]);
          if (s.np > 2 * kWave) ext_add(e, cur.p[2]);
          if (s.nq > 2 * kWave) ext_add(e, cur.q[2]);
        }
        u = meta_of(wave_min4(e));
      }
      // The next pair's loads, in flight while this one is counted.  They
      // follow the use of every vertex in hand: how many they are depends on
      // the pair, so a wait for older loads would wait for them as well.
      int jn = j;
      SweepPair sn = s;
      if (todo) {
        jn = __ffsll((long long)todo) - 1;
        sn = sweep_pair(rec, jn);
        ring_load(sn.p, sn.np, lane, nxt.p);
        if (!kPairBox || sn.q != s.q || sn.nq != s.nq) ring_load(sn.q, sn.nq, lane, nxt.q);
      }
      const bool same_q = kPairBox && sn.q == s.q && sn.nq == s.nq;
      const uint32_t uw = side_u(u.x0, u.x1), uh = side_u(u.y0, u.y1);
      // every coordinate within 2^30: none plus 2^30 above 2^31
      const uint32_t far = max(max((uint32_t)u.x0 + kMaxCoord, (uint32_t)u.x1 + kMaxCoord),
                               max((uint32_t)u.y0 + kMaxCoord, (uint32_t)u.y1 + kMaxCoord));
      const bool ok = far <= 2u * kMaxCoord;
      if (kPairBox && tile_q && on_one_tile(mp)) {
        const bool on_union = union_ok && max(uw, uh) <= (uint32_t)kTile;
        if (on_union || !direct) {
          const uint64_t m = ring_tile(c.slots, lane, cur.p, s.np, mp.x0, mp.y0);
          // column x0 + 63 - L of p is q's lane L + dx, its row r q's row r + dy
          // (tiles that far apart that the difference wraps have none in common)
          const int dx = (int)((uint32_t)mq.x0 - (uint32_t)mp.x0), dy = (int)((uint32_t)mp.y0 - (uint32_t)mq.y0);
          uint64_t t = 0;
          if (max((uint32_t)dx + (kTile - 1), (uint32_t)dy + (kTile - 1)) <= 2u * (kTile - 1)) {
            t = c.slots[kTileQ + dx + lane];
            t = m & (dy >= 0 ? t >> dy : t << -dy);
          }
          uint32_t n, areas;
          if (on_union) {
            const uint32_t both = wave_sum_u32((uint32_t)__popcll(m) | (uint32_t)__popcll(t) << 16);
            n = both >> 16;
            areas = (both & 0xffffu) + pixels_q;
          } else {
            n = wave_pixels(t);
            if (area_q < 0) area_q = ring_area(cur.q, s.nq);
            areas = (uint32_t)(ring_area(cur.p, s.np) + area_q);
          }
          out_i = lane == j ? n : out_i;
          out_u = lane == j ? areas - n : out_u;
          finished |= 1ull << j;
          if (kStats) {
            const unsigned long long nv = (unsigned long long)(s.np + s.nq);
            const Meta box = on_union ? u : pair_box(mp, mq);
            const bool empty = box.x0 >= box.x1 || box.y0 >= box.y1;
            const unsigned long long px = empty ? 0ull : (unsigned long long)side_u(box.x0, box.x1) * side_u(box.y0, box.y1);
            stat_add(c, on_union ? 13 : 12, nv);
            stat_add(c, empty ? 7 : 5, 1ull);
            stat_add(c, 11, px);
            stat_add(c, 1, 1ull);
            stat_add(c, 0, 2ull * px);
            stat_add(c, 10, nv);
            stat_add(c, 14, (unsigned long long)s.np);
          }
        }
      } else if (ok && (!kPairBox || union_ok) && max(uw, uh + 1u) <= (uint32_t)kTile) {
        const uint32_t t = box_count<false>(c.slots, lane, cur, s.np, s.nq, one, u.x0, u.y0, uw, uh);
        if (kPairBox) {
          out_i = lane == j ? t >> 17 : out_i;
          out_u = lane == j ? (t & 0xffffu) - (t >> 17) : out_u;
        } else {
          out_i = lane == j ? t : out_i;
        }
        finished |= 1ull << j;
        if (kStats) {
          const unsigned long long n = (unsigned long long)(s.np + s.nq);
          stat_add(c, 14, n);
          stat_add(c, 5, 1ull);
          stat_add(c, 11, (unsigned long long)uw * uh);
          stat_add(c, 13, n);
          stat_add(c, 1, 1ull);
          stat_add(c, 0, 2ull * (unsigned long long)uw * uh);
          stat_add(c, 10, n);
        }
      } else if (kPairBox && ok && !direct) {
        // the pair box: empty or less than a tile tall, else left to the
        // medium sweep, as is a ring whose area takes 64 bits
        const Meta box = pair_box(mp, mq);
        const bool empty = box.x0 >= box.x1 || box.y0 >= box.y1;
        const uint32_t bw = side_u(box.x0, box.x1), bh = side_u(box.y0, box.y1);
        const bool narrow = side_u(mp.x0, mp.x1) <= (uint32_t)kMaxSide && side_u(mp.y0, mp.y1) <= (uint32_t)kMaxSide &&
                            side_u(mq.x0, mq.x1) <= (uint32_t)kMaxSide && side_u(mq.y0, mq.y1) <= (uint32_t)kMaxSide;
        if (narrow && (empty || max(bw, bh + 1u) <= (uint32_t)kTile)) {
          if (area_q < 0) area_q = ring_area(cur.q, s.nq);
          const uint32_t areas = (uint32_t)(ring_area(cur.p, s.np) + area_q);  // each below 2^30
          uint32_t n = 0;
          if (!empty)
            n = box_count<true>(c.slots, lane, cur, s.np, s.nq, one, box.x0, box.y0, bw, bh) >> 17;
          out_i = lane == j ? n : out_i;
          out_u = lane == j ? areas - n : out_u;
          finished |= 1ull << j;
          if (kStats) {
            const unsigned long long nv = (unsigned long long)(s.np + s.nq);
            stat_add(c, 12, nv);
            stat_add(c, empty ? 7 : 5, 1ull);
            if (!empty) {
              stat_add(c, 11, (unsigned long long)bw * bh);
              stat_add(c, 1, 1ull);
              stat_add(c, 0, 2ull * (unsigned long long)bw * bh);
              stat_add(c, 10, nv);
              stat_add(c, 14, nv);
            }
          }
        }
      }
      s = sn;
      j = jn;
      ring_move(cur.p, nxt.p, s.np);
      if (!same_q) ring_move(cur.q, nxt.q, s.nq);
    }
    if (lane_in(finished)) {
      const uint32_t n = kPairBox ? out_i : out_i >> 17;
      a.inter[i] = (int64_t)n;
      // |p| + |q| - I below 2^31, and below 0 where a ring's loops cancel in its
      // area (no simple ring's do)
      a.uni[i] = kPairBox ? (int64_t)(int32_t)out_u : (int64_t)((out_i & 0xffffu) - n);
    }
    const uint64_t listed = ballot(medium || (sweep && !lane_in(finished)));
    const int st = (int)(blockIdx.x % (unsigned)kStreams);
    if (listed) list_append(a.st->m_count[st].v, a.m_list + st * a.stream_cap, listed, (int32_t)i, lane);
    if (ballot(bucket >= 0)) {
#pragma unroll 1
      for (int b = 0; b < kLptBuckets; ++b) {
        const uint64_t m = ballot(bucket == b);
        if (m) list_append(a.st->p_count[b][st].v, a.l_list + (b * kStreams + st) * a.stream_cap, m, (int32_t)i, lane);
      }
    }
  }
  wave_stamps(a, 0, t_start, lane);
}

// ------------------------------------------------- boxes of several leaf tiles
// A pair box of at most kTileBox leaf tiles is pixelized whole, from one pass
// over each ring per stripe of tiles (most boxes are one stripe), by the
// vertex form of the crossing test (see the union sweep) carried across tiles:
//   - the slots of a stripe hold, per band (64 rows), one 64-bit row mask per
//     column.  A corner XORs the rows of its own band at or above it into its
//     column's slot of that band only: one LDS atomic per vertex, however tall
//     the box is.  In the bands above it the corner toggles every row, which
//     the scan recovers by itself: the top row of a column's parities in one
//     band is what the rows of the next band start from.
//   - a lane owns `cols` neighbouring columns of a band (cols = the stripe's
//     width in tiles), so that one 64-lane scan serves the whole row: it XORs
//     its columns up, the lanes scan their totals, and each column takes the
//     scan's offset and the carry from the band below.  Per 64x64 tile and
//     ring that is about 7 + 14 / cols vector instructions; a scan per tile
//     took 24 and its carries.
//   - corners left of the stripe toggle none of its columns, those right of
//     it all of them; those below it count as standing in its first row, those
//     above it not at all.  So stripes are independent of each other, and a
//     pixel of the last tiles past the pair box lies outside MBR(p) or MBR(q)
//     and adds nothing to the intersection.
// Column k of lane L stands at position L cols + k from the right and at slot
// (band cols + k) 64 + L, which every lane reads without bank conflicts.
// Measured: 8191 pairs of merged blobs (530 vertices a ring, boxes of about
// 4 x 4 tiles) 1562 -> 76 us and 15,724 five-fold scaled pairs 561 -> 51 us,
// against tiles scattered one by one, or a band row at a time, from rings
// streamed anew for each.
constexpr int kTileBox = 64;   // most leaf tiles of a box pixelized this way
constexpr int kMaxCols = 8;    // widest stripe, in tiles
// A box is classified instead (Lemma 1, in the persistent kernel) when the
// caller asks for it from fewer tiles than the default.
constexpr int kDefaultClassifyCells = 26;
__device__ __forceinline__ bool tile_box(const BatchArgs& a, int gx, int gy) {
  const int t = gx * gy;
  return t == 1 || (t <= kTileBox && (t < a.min_classify_cells || a.min_classify_cells >= kDefaultClassifyCells));
}

// Extents, doubled area and corners of a ring of nr (>= 1) vertices held in N
// chunks of 64 (lanes past the end hold the last vertex again).  f: its first
// vertex; carry: whether the closing edge is vertical.  tn gains twice the signed area, summed as (x + x') (y' - y) over the edges with x
// relative to f, modulo 2^32: exact for a ring at most kMaxSide wide and
// tall.  Returns the corners, vertices with exactly one vertical edge: bit c
// for the lane's vertex of chunk c (kept per lane: N wave-wide masks are more
// scalar registers than there are).
template <int N>
__device__ __forceinline__ uint32_t ring_pass(const int2 (&d)[N], int nr, int lane, int2 f, uint32_t carry, Ext& e,
                                              uint32_t& tn) {
  uint32_t corners = 0;
  const int nc = (nr + kWave - 1) / kWave, le = (nr - 1) & (kWave - 1);
#pragma unroll
  for (int c = 0; c < N; ++c) {
    if (c < nc) {
      const bool last = c == nc - 1;
      const int2 n0 = lane_value(d[c + 1 < N ? c + 1 : c], 0);
      const int2 nx = last ? f : n0;
      int sx = __builtin_amdgcn_update_dpp(nx.x, d[c].x, 0x130, 0xf, 0xf, false);  // the next lane's
      int sy = __builtin_amdgcn_update_dpp(nx.y, d[c].y, 0x130, 0xf, 0xf, false);
      if (last && le != kWave - 1) {
        // past the end: edges of no length
        sx = lane == le ? f.x : lane > le ? d[c].x : sx;
        sy = lane == le ? f.y : lane > le ? d[c].y : sy;
      }
      const uint64_t b = ballot(d[c].x == sx);
      corners |= lane_in((b ^ ((b << 1) | carry)) & (last ? ~0ull >> (kWave - 1 - le) : ~0ull)) ? 1u << c : 0u;
      carry = (uint32_t)(b >> (kWave - 1));
      ext_add(e, d[c]);
      tn += (uint32_t)__mul24((int)((uint32_t)d[c].x + (uint32_t)sx - 2u * (uint32_t)f.x),
                              (int)((uint32_t)sy - (uint32_t)d[c].y));
    }
  }
  return corners;
}

// |shoelace|/2 of a ring wider or taller than kMaxSide, streamed: summed
// modulo 2^64, in which twice the area (at most 2^63 in size) is exact.
__device__ __forceinline__ int64_t ring_area_wide(const int2* xy, int64_t o, int nv, int lane) {
  uint64_t tw = 0;
  RingStream rs(xy, o, nv, lane);
#pragma unroll 1
  do {
    rs.ahead();
    const int2 w = rs.succ();
    if (rs.valid()) tw += (uint64_t)((int64_t)rs.cur.x * w.y) - (uint64_t)((int64_t)w.x * rs.cur.y);
  } while (rs.next());
  const uint64_t t = wave_sum_u64(tw);
  return (int64_t)(((int64_t)t < 0 ? 0 - t : t) / 2);
}

// Extent and area of a non-empty ring from its lanes' extents and doubled
// areas (see ring_pass), which are summed again if a side exceeds `narrow`.  A
// ring with a coordinate beyond 2^30 sets `bad` and covers nothing.
__device__ __forceinline__ void ring_meta(const int2* xy, int64_t o, int nv, int lane, const Ext& lanes, uint32_t tn,
                                          uint32_t narrow, Meta& m, int64_t& area, bool& bad) {
  m = meta_of(wave_min4(lanes));
  bad = out_of_range(m);
  if (bad) {
    m = Meta{INT_MAX, INT_MAX, INT_MIN, INT_MIN};
    area = 0;
  } else if (max(side_u(m.x0, m.x1), side_u(m.y0, m.y1)) <= narrow) {
    const int32_t t = (int32_t)wave_sum_u32(tn);
    area = (t < 0 ? -(int64_t)t : (int64_t)t) / 2;
  } else {
    area = ring_area_wide(xy, o, nv, lane);
  }
}

// A stripe of tiles: `cols` tiles wide from x0, `bands` of 64 rows from y0.
struct Stripe {
  int x0, y0, cols, bands;
  uint32_t inv;  // ceil(2^16 / cols): position / cols = (position inv) >> 16 below 512
};

// XOR the end (x, y) of a vertical edge into the stripe's slots, when `take`.
__device__ __forceinline__ void stripe_xor(uint64_t* slots, int2 v, bool take, const Stripe& s) {
  const int wpad = s.cols * kTile, sh = s.bands * kTile;
  const int dx = min(v.x, s.x0 + wpad) - s.x0;
  const int ty = max(min(v.y, s.y0 + sh) - s.y0, 0);
  const uint32_t pos = (uint32_t)(wpad - dx);
  const uint32_t q = __umul24(pos, s.inv) >> 16;
  const uint32_t at = __umul24((uint32_t)ty >> 6, (uint32_t)wpad) + (pos << 6) - __umul24(q, (uint32_t)(wpad - 1));
  if (take & (dx > 0) & (ty < sh)) slot_xor(slots, (int)at, ~0ull << (ty & 63));
}
// The corners of a ring in registers (see ring_pass).
template <int N>
__device__ __forceinline__ void stripe_scatter(uint64_t* slots, const int2 (&d)[N], uint32_t corners, int nr,
                                               const Stripe& s) {
  // made anew for each stripe: tests of the chunks and corners that the
  // compiler hoists out of the stripes' loop are dozens of spilled registers
  asm volatile("" : "+v"(corners), "+s"(nr));
#pragma unroll
  for (int c = 0; c < N; ++c)
    if (c * kWave < nr) stripe_xor(slots, d[c], (corners >> c) & 1u, s);
}
// A longer ring, streamed: both ends of every vertical edge.
__device__ __forceinline__ void stripe_stream(uint64_t* slots, const int2* xy, int64_t o, int nv, int lane,
                                              const Stripe& s) {
  RingStream rs(xy, o, nv, lane);
#pragma unroll 1
  do {
    rs.ahead();
    const int2 w = rs.succ();
    const bool vertical = rs.valid() && rs.cur.x == w.x;
    stripe_xor(slots, rs.cur, vertical, s);
    stripe_xor(slots, w, vertical, s);
  } while (rs.next());
}

// The scan of one band of one ring: what every column of the lane takes from
// the lanes right of it.  The columns' slots are read twice, here and by the
// caller: held in registers they cost the kernel a wave per SIMD.
template <int C>
__device__ __forceinline__ uint64_t band_offset(const uint64_t* s, int lane) {
  uint64_t t = s[lane];
#pragma unroll
  for (int k = 1; k < C; ++k) t ^= s[k * kWave + lane];
  t ^= wave_prefix_xor<false>(t);
  asm volatile("" ::: "memory");  // or the compiler keeps the slots in registers after all
  return t;
}
// A column's parities from the slots up to it and its carry, which holds all
// ones when the row below the band is inside, and then the band's top row.
__device__ __forceinline__ uint64_t column_parities(uint64_t run, uint32_t& carry) {
  const uint32_t lo = (uint32_t)run ^ carry, hi = (uint32_t)(run >> 32) ^ carry;
  carry = (uint32_t)((int32_t)hi >> 31);
  return ((uint64_t)hi << 32) | lo;
}

// A lane's share of the pixels inside both rings, from both rings' slots.
template <int C>
__device__ __forceinline__ uint32_t stripe_count(const uint64_t* sp, const uint64_t* sq, int bands, int lane) {
  uint32_t cp[C] = {}, cq[C] = {}, n = 0;
#pragma unroll 1
  for (int j = 0; j < bands; ++j, sp += C * kWave, sq += C * kWave) {
    uint64_t p = band_offset<C>(sp, lane), q = band_offset<C>(sq, lane);
#pragma unroll
    for (int k = 0; k < C; ++k) {
      p ^= sp[k * kWave + lane];
      q ^= sq[k * kWave + lane];
      n += (uint32_t)__popcll(column_parities(p, cp[k]) & column_parities(q, cq[k]));
    }
  }
  return n;
}
// One ring's slots turned into parities in place.
template <int C>
__device__ __forceinline__ void stripe_scan(uint64_t* s, int bands, int lane) {
  uint32_t carry[C] = {};
#pragma unroll 1
  for (int j = 0; j < bands; ++j, s += C * kWave) {
    uint64_t t = band_offset<C>(s, lane);
#pragma unroll
    for (int k = 0; k < C; ++k) {
      t ^= s[k * kWave + lane];
      s[k * kWave + lane] = column_parities(t, carry[k]);
    }
  }
}
#define SCCG_BY_COLS(cols, CALL) \
  switch (cols) {                \
    case 1: CALL(1); break;      \
    case 2: CALL(2); break;      \
    case 3: CALL(3); break;      \
    case 4: CALL(4); break;      \
    case 5: CALL(5); break;      \
    case 6: CALL(6); break;      \
    case 7: CALL(7); break;      \
    default: CALL(8); break;     \
  }

// Calls f(stripe) for the stripes of a box gx x gy tiles large, with room for
// `cap` tiles and at most `most` columns each.
template <typename F>
__device__ __forceinline__ void for_stripes(const Meta& box, int gx, int gy, int cap, int most, F f) {
  const int nx = (gx + most - 1) / most, cols = (gx + nx - 1) / nx;
  const int bands = min(cap / cols, gy);
#pragma unroll 1
  for (int x = 0; x < gx; x += cols) {
    const int w = min(cols, gx - x);
#pragma unroll 1
    for (int y = 0; y < gy; y += bands)
      f(Stripe{box.x0 + x * kTile, box.y0 + y * kTile, w, min(bands, gy - y),
               (uint32_t)((65536 + w - 1) / w)});
  }
}

// The intersection counted on a pair box of one leaf tile, from rings whose
// corners are known (as box_count with clipping).  kHalves: the box is at most 32 wide,
// p's columns in lanes 0-31 and q's in 32-63; M: 32-bit rows when it is at
// most 32 tall.
template <bool kHalves, typename M, int N>
__device__ __forceinline__ uint32_t corner_count(uint64_t* slot_words, const int2 (&p)[N], uint32_t cp, int np,
                                                 const int2 (&q)[N], uint32_t cq, int nq, const Meta& box, int lane) {
  constexpr int W = kHalves ? 32 : kWave, R = (int)sizeof(M) * 8;
  M* slots = reinterpret_cast<M*>(slot_words);
  slots[lane] = (M)0;
  if (!kHalves) slots[kWave + lane] = (M)0;
  wave_sync_lds();
  auto scatter = [&](const int2(&d)[N], uint32_t corners, int nr, int base) {
#pragma unroll
    for (int c = 0; c < N; ++c) {
      if (c * kWave < nr) {
        const int dx = min(d[c].x, box.x0 + W) - box.x0;
        const int ty = max(min(d[c].y, box.y0 + R) - box.y0, 0);
        if ((((corners >> c) & 1u) != 0u) & (dx > 0) & (ty < R)) slot_xor(slots + base + W - dx, 0, (M)(~(M)0 << ty));
      }
    }
  };
  scatter(p, cp, np, 0);
  scatter(q, cq, nq, W);
  wave_sync_lds();
  uint32_t n;
  if (kHalves) {
    const M m = wave_prefix_xor<true>(slots[lane]);
    const M o = upper_half(m);
    n = lane < 32 ? (uint32_t)__popcll((uint64_t)(m & o)) : 0u;
  } else {
    n = (uint32_t)__popcll((uint64_t)(wave_prefix_xor<false>(slots[lane]) & wave_prefix_xor<false>(slots[kWave + lane])));
  }
  wave_sync_lds();
  return n;
}

// ------------------------------------------------------------ medium sweep
// Second pass, two kinds of pairs:
//   - the long pairs the sweep listed (a ring over kMediumRing vertices,
//     or at least heavy_verts in all), largest bucket first, two waves per
//     pair, one per ring: each loads its ring (kLongChunks chunks at once),
//     reduces its MBR and area, scatters and scans its own slots without
//     waiting for the other, and both count the tiles; two barriers per
//     stripe.
//   - then the medium list: pairs with rings of at most kMediumRing vertices
//     that the union sweep did not finish (a ring over kSweepRing vertices or
//     an empty one, or a union box larger than a leaf tile), one wave per
//     pair, rings in registers.
// Both pixelize boxes of up to kTileBox tiles at once; a larger one, one to be
// classified, or any one when the union is counted directly, is listed with
// its box for the persistent kernel, I = 0 and U = |p| + |q| (0 when the union
// is counted directly) as the values its boxes add to.
// Bound by instruction issue; five waves per SIMD with 14 tiles of slots per
// ring: four (with 18 tiles) or six (12 tiles, registers spilled) were 3 to 5 %
// slower on the heavy-tailed mix.
constexpr int kTeamWaves = 2;    // waves per workgroup: one pair's team, or two waves with a pair each
constexpr int kLongChunks = 16;  // chunks of a long ring in registers; a longer ring is taken in parts
constexpr int kTeamTiles = SCCG_TEAM_TILES;   // tiles per ring and stripe of a team
constexpr int kWaveTiles = kTeamTiles / 2;   // tiles per ring and stripe of a single wave
static_assert(2 * kWaveTiles <= kTeamTiles && kMaxCols <= kTeamTiles, "the team's slots hold either kind's stripes");

// What the two waves of a team tell each other of their rings.
struct TeamRing {
  Meta m;
  int64_t area;
  int32_t nv, bad;
};

// List the pairs i of the lanes `m`, of `verts` vertices each, for the
// persistent kernel: one append per bucket, to the workgroup's stream (on one
// counter an append took 25 ns: 400 us for 16,000 pairs that were all listed one
// by one; of 3000 pairs a wave each and 10,000 in 5120 waves, appended a wave's
// at a time, the medium sweep took 96 and 155 us, on a counter per stream 32 and
// 37, and the persistent kernel, which reads them all, no longer).
// The arguments are read again where they are needed, from the kernel's own: in
// registers throughout they were 42 more spilled scalars in the loops around.
__device__ __forceinline__ void list_run(uint64_t m, int32_t i, int64_t verts, int lane) {
  typedef const BatchArgs __attribute__((address_space(4))) * args_ptr;
  args_ptr a = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();  // the kernel's only parameter
  asm volatile("" : "+s"(a));
  const int st = (int)(blockIdx.x % (unsigned)kStreams);
  const int bucket = lpt_bucket(a->flags, a->heavy_verts, verts);
#pragma unroll 1
  for (int b = 0; b < kLptBuckets; ++b) {
    const uint64_t mb = m & ballot(bucket == b);
    if (mb) list_append(a->st->l_count[st].v[b], a->run_list + (int64_t)(b * kStreams + st) * a->run_cap, mb, i, lane);
  }
}
// A listed pair's box and class (by one lane).
__device__ __forceinline__ void listed_pair(const BatchArgs& a, int64_t i, const Meta& box, uint8_t cls) {
  *reinterpret_cast<int4*>(a.hbox + i) = make_int4(box.x0, box.y0, box.x1, box.y1);
  a.cls[i] = cls;
}

// Every chunk of both rings of a medium pair (clamped to each ring's last
// vertex), or for no pair or an empty ring reads of `dummy`.
__device__ __forceinline__ void medium_load(const BatchArgs& a, const PairRec& s, int lane, PairRegs<kMediumChunks>& r) {
  const int2* dummy = reinterpret_cast<const int2*>(a.st);
  const int2* P = s.np > 0 ? a.A.xy + s.op : dummy;
  const int2* Q = s.nq > 0 ? a.B.xy + s.oq : dummy;
  const int lp = max(s.np - 1, 0), lq = max(s.nq - 1, 0);
#pragma unroll
  for (int c = 0; c < kMediumChunks; ++c) {
    r.p[c] = P[min(c * kWave + lane, lp)];
    r.q[c] = Q[min(c * kWave + lane, lq)];
  }
}

// What a pair's MBRs and areas make of it: its class, its box and the counts
// it has before any box is counted.  kClsDone: I and U are final.
__device__ __forceinline__ uint8_t pair_class(Ctx& c, const Meta& mp, const Meta& mq, int64_t areas, int64_t verts,
                                              bool bad, bool tell, int64_t& U, Meta& box) {
  const BatchArgs& a = *c.a;
  if (tell && bad && c.lane == 0) latch_error(a.err, kErrCoord);
  const bool direct = direct_union(a);
  box = direct ? union_box(mp, mq) : pair_box(mp, mq);
  U = direct ? 0 : areas;
  if (tell) stat_add(c, 12, (unsigned long long)verts);
  const bool empty = box.x0 >= box.x1 || box.y0 >= box.y1;
  const uint32_t bw = side_u(box.x0, box.x1), bh = side_u(box.y0, box.y1);
  const bool wide = !empty && (bw > (uint32_t)kMaxSide || bh > (uint32_t)kMaxSide);
  if (wide) {
    if (tell && c.lane == 0) latch_error(a.err, kErrSide);
    U = 0;
  }
  if (empty || wide) return kClsDone;
  const bool small = bw <= (uint32_t)kTile && bh <= (uint32_t)kTile;
  if (tell) {
    stat_add(c, small ? 5 : 6, 1ull);
    stat_add(c, 11, (unsigned long long)bw * bh);
  }
  return small ? kClsSmall : kClsLarge;
}

// Returns whether the pair is to be listed for the persistent kernel.
__device__ __forceinline__ bool medium_one(Ctx& c, const PairRec& s, const PairRegs<kMediumChunks>& r, int64_t i) {
  const BatchArgs& a = *c.a;
  const int lane = c.lane;
  Meta mp{INT_MAX, INT_MAX, INT_MIN, INT_MIN}, mq = mp, box;
  int64_t ap = 0, aq = 0, I = 0, U = 0;
  bool bp = false, bq = false;
  auto meta = [&](const int2(&d)[kMediumChunks], const int2* xy, int64_t o, int nv, Meta& m, int64_t& area,
                  bool& bad) -> uint32_t {
    if (nv <= 0) return 0;
    Ext e = ext_of(d[0]);
    const int2 f = lane_value(d[0], 0);
    // every chunk is loaded, so the last lane of the last one holds the last vertex
    uint32_t tn = 0;
    const uint32_t carry = __builtin_amdgcn_readlane(d[kMediumChunks - 1].x, kWave - 1) == f.x ? 1u : 0u;
    const uint32_t corners = ring_pass<kMediumChunks>(d, nv, lane, f, carry, e, tn);
    ring_meta(xy, o, nv, lane, e, tn, kMaxSide, m, area, bad);
    return corners;
  };
  const uint32_t cp = meta(r.p, a.A.xy, s.op, s.np, mp, ap, bp);
  const uint32_t cq = meta(r.q, a.B.xy, s.oq, s.nq, mq, aq, bq);
  const uint8_t cls = pair_class(c, mp, mq, ap + aq, (int64_t)s.np + s.nq, bp || bq, true, U, box);
  bool listed = false;
  if (cls == kClsDone) {
    stat_add(c, 7, 1ull);  // an empty or rejected box: nothing in common
  } else {
    const int gx = (box.x1 - box.x0 + kTile - 1) / kTile, gy = (box.y1 - box.y0 + kTile - 1) / kTile;
    if (direct_union(a) || !tile_box(a, gx, gy)) {
      listed = true;
    } else {
      uint32_t n = 0, passes = 0;
      const int bw = box.x1 - box.x0, bh = box.y1 - box.y0;
      if (gx * gy == 1) {
        passes = 1;
#define SCCG_CORNERS(HALVES, M) corner_count<HALVES, M>(c.slots, r.p, cp, s.np, r.q, cq, s.nq, box, lane)
        if (bw <= 32)
          n = bh <= 32 ? SCCG_CORNERS(true, uint32_t) : SCCG_CORNERS(true, uint64_t);
        else
          n = bh <= 32 ? SCCG_CORNERS(false, uint32_t) : SCCG_CORNERS(false, uint64_t);
#undef SCCG_CORNERS
      } else {
        for_stripes(box, gx, gy, kWaveTiles, min(kWaveTiles, kMaxCols), [&](const Stripe& st) {
          uint64_t* sp = c.slots;
          uint64_t* sq = c.slots + st.cols * st.bands * kTile;
#pragma unroll 1
          for (int t = 0; t < 2 * st.cols * st.bands; ++t) sp[t * kWave + lane] = fresh_zero<uint64_t>();
          wave_sync_lds();
          stripe_scatter(sp, r.p, cp, s.np, st);
          stripe_scatter(sq, r.q, cq, s.nq, st);
          wave_sync_lds();
#define SCCG_COUNT(C) n += stripe_count<C>(sp, sq, st.bands, lane)
          SCCG_BY_COLS(st.cols, SCCG_COUNT)
#undef SCCG_COUNT
          wave_sync_lds();
          passes += 1;
        });
      }
      I = (int64_t)wave_sum_u32(n);
      if (c.stats) {
        stat_add(c, 1, (unsigned long long)gx * gy);
        stat_add(c, 0, 2ull * (unsigned long long)bw * bh);
        stat_add(c, 10, (unsigned long long)(s.np + s.nq) * passes);
        stat_add(c, 14, (unsigned long long)(s.np + s.nq) * passes);
      }
    }
  }
  if (lane == 0) {
    a.inter[i] = I;
    a.uni[i] = U - I;
    if (listed) listed_pair(a, i, box, cls);
  }
  return listed;
}

// One long pair, both waves of the team (wave w has ring w).  Returns as
// medium_one does.
template <bool kStats>
__device__ __forceinline__ bool long_one(Ctx& c, int64_t i, int w, uint64_t* team_slots, TeamRing* ex) {
  const BatchArgs& a = *c.a;
  const int lane = c.lane;
  const int2* xy = w ? a.B.xy : a.A.xy;
  const int64_t* off = (w ? a.B.off + a.pb[i] : a.A.off + a.pa[i]);
  const int64_t o = uniform64(off[0]);
  const int nv = uniform((int)(off[1] - o));
  const int2* R = xy + o;
  uint64_t* slots = team_slots + w * kTeamTiles * kTile;
  int2 d[kLongChunks];
  const bool held = nv <= kLongChunks * kWave;
  Meta m{INT_MAX, INT_MAX, INT_MIN, INT_MIN};
  int64_t area = 0;
  bool bad = false;
  uint32_t corners = 0;
  if (nv > 0) {
    Ext e{INT_MAX, INT_MAX, INT_MAX, INT_MAX};
    uint32_t tn = 0;
    if (held) {
#pragma unroll
      for (int q = 0; q < kLongChunks; ++q)
        if (q * kWave < nv) d[q] = R[min(q * kWave + lane, nv - 1)];
      const int x_last = uniform(R[nv - 1].x);
      const int2 f = lane_value(d[0], 0);
      corners = ring_pass<kLongChunks>(d, nv, lane, f, x_last == f.x ? 1u : 0u, e, tn);
    } else {
      RingStream rs(xy, o, nv, lane);
      const int2 f = rs.first;
#pragma unroll 1
      do {
        rs.ahead();
        const int2 v = rs.cur, x = rs.succ();
        ext_add(e, v);
        const uint32_t t = (uint32_t)__mul24((int)((uint32_t)v.x + (uint32_t)x.x - 2u * (uint32_t)f.x),
                                             (int)((uint32_t)x.y - (uint32_t)v.y));
        tn += rs.valid() ? t : 0u;
      } while (rs.next());
    }
    // sides from 2^14 on in 64 bits: a long ring may run around its pixels often
    ring_meta(xy, o, nv, lane, e, tn, (1u << 14) - 1u, m, area, bad);
  }
  if (lane == 0) ex[w] = TeamRing{m, area, nv, bad ? 1 : 0};
  __syncthreads();
  const TeamRing rp = ex[0], rq = ex[1];
  Meta box;
  int64_t U = 0;
  const int64_t verts = (int64_t)uniform(rp.nv) + uniform(rq.nv);
  const uint8_t cls = pair_class(c, rp.m, rq.m, rp.area + rq.area, verts, (rp.bad | rq.bad) != 0, w == 0, U, box);
  box = Meta{uniform(box.x0), uniform(box.y0), uniform(box.x1), uniform(box.y1)};
  const int gx = (box.x1 - box.x0 + kTile - 1) / kTile, gy = (box.y1 - box.y0 + kTile - 1) / kTile;
  const bool settled = uniform(cls) == kClsDone;
  if (settled && w == 0) stat_add(c, 7, 1ull);
  const bool listed = !settled && (direct_union(a) || !tile_box(a, gx, gy));
  uint32_t n = 0;
  if (!settled && !listed) {
    uint32_t passes = 0;
    for_stripes(box, gx, gy, kTeamTiles, kMaxCols, [&](const Stripe& st) {
      const int tiles = st.cols * st.bands;
#pragma unroll 1
      for (int t = 0; t < tiles; ++t) slots[t * kWave + lane] = fresh_zero<uint64_t>();
      wave_sync_lds();
      if (nv > 0) {
        if (held)
          stripe_scatter(slots, d, corners, nv, st);
        else
          stripe_stream(slots, xy, o, nv, lane, st);
      }
      wave_sync_lds();
#define SCCG_SCAN(C) stripe_scan<C>(slots, st.bands, lane)
      SCCG_BY_COLS(st.cols, SCCG_SCAN)
#undef SCCG_SCAN
      __syncthreads();
#pragma unroll 1
      for (int t = w * kWave + lane; t < tiles * kTile; t += kTeamWaves * kWave)
        n += (uint32_t)__popcll(team_slots[t] & team_slots[kTeamTiles * kTile + t]);
      __syncthreads();
      passes += 1;
    });
    n = wave_sum_u32(n);
    if (kStats) {
      stat_add(c, 14, (unsigned long long)nv * passes);
      stat_add(c, 10, (unsigned long long)nv * passes);
      if (w == 0) {
        stat_add(c, 1, (unsigned long long)gx * gy);
        stat_add(c, 0, 2ull * (unsigned long long)(box.x1 - box.x0) * (unsigned long long)(box.y1 - box.y0));
      }
    }
    // wave 1's share reaches wave 0 through its entry of the exchange
    if (w == 1 && lane == 0) ex[1].nv = (int)n;
    __syncthreads();
    n += w == 0 ? (uint32_t)uniform(ex[1].nv) : 0u;
  }
  if (w == 0 && lane == 0) {
    a.inter[i] = (int64_t)n;
    a.uni[i] = U - (int64_t)n;
    if (listed) listed_pair(a, i, box, cls);
  }
  return listed;
}

template <bool kStats>
__global__ void __launch_bounds__(kTeamWaves* kWave) __attribute__((amdgpu_waves_per_eu(SCCG_MEDIUM_WAVES_PER_EU)))
k_batch_medium(BatchArgs args) {
  __shared__ __align__(16) uint64_t team_slots[2 * kTeamTiles * kTile];
  __shared__ TeamRing ex[2][2];
  __shared__ int64_t claimed[2];
  const int w = uniform((int)(threadIdx.x / kWave));
  Ctx c;
  c.a = &args;
  c.stats = kStats;
  c.lane = lane_id();
  c.slots = team_slots + w * 2 * kWaveTiles * kTile;
  c.local = nullptr;
  c.lsp = 0;
  c.home = 0;
  c.xcd = (int)(blockIdx.x % (unsigned)kStreams);
  const BatchArgs& a = args;
  const int lane = c.lane;
  const unsigned long long t_start = wave_stamp(a);
  if (blockIdx.x == 0 && threadIdx.x < (unsigned)kMaxGrid) {
    // the queues of the previous call were cleared by the sweep
    a.st->q_head[threadIdx.x].v = 0;
    a.st->q_tail[threadIdx.x].v = 0;
  }
  const uint32_t own = gridDim.x < (unsigned)kStreams ? 0u : (0xffu & ~(1u << c.xcd));
  uint32_t p_empty = own;
  // the long pairs, bucket after bucket from the largest, one pair per claim;
  // wave 0 claims the next one while the team works on the one in hand
  // the lengths of these lists and, in the lanes after them, of the medium
  // list's parts, in one load
  static_assert(kParts + kStreams <= kWave, "a list per lane");
  const int length = lane < kParts              ? (int)a.st->p_count[BucketLists::bucket(lane)][lane % kStreams].v
                     : lane < kParts + kStreams ? (int)a.st->m_count[lane - kParts].v
                                                : 0;
  if (!ballot(length != 0)) {
    wave_stamps(a, 1, t_start, lane);
    return;  // both waves of the team
  }
  const BucketLists longs(lane < kParts ? length : 0, lane);
  const int64_t n_long = longs.all;
  if (n_long > 0) {
    // wave 0's lanes keep the pairs to be listed
    int32_t listed = 0;
    int n_listed = 0;
    auto list_long = [&]() {
      const bool mine = lane < n_listed;
      int64_t verts = 0;
      if (mine) {
        const PairRec r = pair_rec(a, a.pa[listed], a.pb[listed]);
        verts = (int64_t)r.np + r.nq;
      }
      list_run(ballot(mine), listed, verts, lane);
      n_listed = 0;
    };
    int64_t next = -1;
    if (w == 0) next = claim_chunk(a.st->p_next, n_long, 1, c.xcd, lane, p_empty);
#pragma unroll 1
    for (int it = 0;; it ^= 1) {
      if (w == 0) {
        if (lane == 0) claimed[it] = next;
        if (next >= 0) next = claim_chunk(a.st->p_next, n_long, 1, c.xcd, lane, p_empty);
      }
      __syncthreads();
      const int64_t k = uniform64(claimed[it]);
      if (k < 0) break;
      const int64_t i = a.l_list[longs.at(k, a.stream_cap, lane)];
      if (long_one<kStats>(c, uniform64(i), w, team_slots, ex[it]) && w == 0) {
        listed = lane == n_listed ? (int32_t)i : listed;
        if (++n_listed == kWave) list_long();
      }
    }
    if (n_listed > 0) list_long();
    __syncthreads();
  }
  // the medium list, its streams' parts end to end
  ListParts parts;
  parts.of_lanes(length, kParts);
  // every wave takes an equal share of the list, single entries dealt out in
  // turns over the waves: the pairs are alike enough, and a
  // claim per few entries left each wave waiting on a counter, the list, the
  // records and the rings in turn (200,000 uniform pairs, 26,000 of them here:
  // 74 us with claims)
  const WaveShare share(parts.total, kTeamWaves, w, 1);
#pragma unroll 1
  for (uint32_t k0 = 0; k0 < share.count; k0 += kWave) {
    const int cnt = uniform((int)min((uint32_t)kWave, share.count - k0));
    // lane j: pair index and record of the wave's entry k0 + j
    int idx = 0;
    PairRec recs{0, 0, 0, 0};
    if (lane < cnt) {
      idx = a.m_list[parts.at(share.entry(k0 + (uint32_t)lane), a.stream_cap)];
      recs = pair_rec(a, a.pa[idx], a.pb[idx]);
    }
    // the pair in hand (sc, rc) and the next one (sn, rn), whose loads are in
    // flight while the pair in hand is processed: every chunk of both rings,
    // loaded the same way whatever the pair, so that the compiler waits only
    // for the pair in hand's loads
    PairRegs<kMediumChunks> rc, rn;
    PairRec sc = rec_of_lane(recs, 0);
    uint64_t listed = 0;
    medium_load(a, sc, lane, rc);
#pragma unroll 1
    for (int j = 0; j < cnt; ++j) {
      const PairRec sn = j + 1 < cnt ? rec_of_lane(recs, j + 1) : PairRec{0, 0, 0, 0};
      medium_load(a, sn, lane, rn);
      if (medium_one(c, sc, rc, (int64_t)__builtin_amdgcn_readlane(idx, j))) listed |= 1ull << j;
      sc = sn;
      rc = rn;
    }
    if (listed) list_run(listed, idx, (int64_t)recs.np + recs.nq, lane);
  }
  wave_stamps(a, 1, t_start, lane);
}

// ----------------------------------------------------------- persistent run
// Third pass: the pairs the medium sweep listed, each with its box: those of
// more leaf tiles than it counts at once, those to be classified, and every
// pair of more than one when the union is counted directly.  Waves claim, in
// this order: boxes from their queue, listed pairs, boxes from any queue.
template <bool kStats>
__global__ void __launch_bounds__(512) SCCG_RUN_ATTR k_batch_run(BatchArgs args) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int wave = threadIdx.x / kWave;
  Ctx c;
  c.a = &args;
  c.stats = kStats;
  c.lane = lane_id();
  unsigned char* lds = smem + (size_t)wave * kLdsPerWave;
  c.slots = reinterpret_cast<uint64_t*>(lds);
  c.local = reinterpret_cast<uint64_t*>(lds + kRowSlotsPerWave * 8);
  c.lsp = 0;
  c.xcd = (int)(blockIdx.x % (unsigned)kStreams);
  c.home = c.xcd % args.n_queues;
  const BatchArgs& a = args;
  const unsigned long long t_start = wave_stamp(a);
  if (blockIdx.x == 0) {
    // the lists that the next call's sweep appends to (see next_call_state)
    for (unsigned t = threadIdx.x; t < (unsigned)((kLptBuckets + 1) * kStreams); t += blockDim.x) {
      if (t < (unsigned)(kLptBuckets * kStreams))
        a.st->p_count[t / kStreams][t % kStreams].v = 0;
      else
        a.st->m_count[t % kStreams].v = 0;
    }
  }
  const int length = c.lane < kParts ? (int)a.st->l_count[c.lane % kStreams].v[BucketLists::bucket(c.lane)] : 0;
  if (!ballot(length != 0)) {
    wave_stamps(a, 2, t_start, c.lane);
    return;
  }
  const BucketLists lists(length, c.lane);
  // Boxes reach a queue only from splits with at least min_cells_to_queue
  // continuing cells (at most 64): otherwise no wave ever needs to look at
  // the queues.
  const bool queues_used = !(a.flags & SCCG_F_NO_SPLIT_QUEUE) && a.min_cells_to_queue <= kWave;
  // streams of the lists found exhausted (wave-uniform); as in the sweeps, a
  // wave claims only from its XCD's stream unless kRunSteal
  uint32_t l_empty = kRunSteal || gridDim.x < (unsigned)kStreams ? 0u : (0xffu & ~(1u << c.xcd));
  for (;;) {
    PairInfo pi;
    uint64_t task = 0;  // 0: a box that fits one leaf tile
    uint64_t w;
    bool have = false;
    if (queues_used && queue_claim(c, false, &w)) {
      pi = heavy_info(a, task_decode(w).hidx);
      task = w;
      have = true;
    }
    if (!have) {
      const int64_t e = claim_chunk(a.st->l_next, lists.all, 1, c.xcd, c.lane, l_empty);
      if (e >= 0) {
        pi = heavy_info(a, (int64_t)a.run_list[lists.at(e, a.run_cap, c.lane)]);
        if (a.cls[pi.pair] == kClsLarge) task = root_task(pi);
        have = true;
      }
    }
    // nothing of its own left: help with every queue, then stop
    if (!have) {
      if (!queues_used || !queue_claim(c, true, &w)) break;
      pi = heavy_info(a, task_decode(w).hidx);
      task = w;
    }
    uint64_t I;
    if (task == 0)
      I = leaf_count(c, pi, pi.box.x0, pi.box.y0, pi.box.x1 - pi.box.x0, pi.box.y1 - pi.box.y0, false, false);
    else
      I = run_large(c, pi, task);
    if (c.lane == 0) add_counts(a, pi.pair, I);
  }
  wave_stamps(a, 2, t_start, c.lane);
}

// ------------------------------------------------------------------ launches
__global__ void k_batch_clear_stats(BatchState* st) {
  if (threadIdx.x < (unsigned)kNumStats) st->stats[threadIdx.x] = 0;
}

int batch_occupancy(int waves_per_wg) {
  int n = 0;
  const size_t lds = (size_t)waves_per_wg * batch_lds_bytes_per_wave();
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_run<false>, waves_per_wg * kWave, lds) != hipSuccess)
    return 1;
  return n > 0 ? n : 1;
}

int batch_sweep_occupancy(bool pair_box) {
  int n = 0;
  const hipError_t e =
      pair_box ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_sweep<true, false>, kSweepWaves * kWave, 0)
               : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_sweep<false, false>, kSweepWaves * kWave, 0);
  return e == hipSuccess && n > 0 ? n : 1;
}

int batch_medium_occupancy() {
  int n = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_medium<false>, kTeamWaves * kWave, 0);
  return e == hipSuccess && n > 0 ? n : 1;
}

int batch_sweep_waves_per_wg() { return kSweepWaves; }
int batch_medium_waves_per_wg() { return kTeamWaves; }

hipError_t launch_batch_sweeps(const BatchArgs& a, int sweep_grid, int medium_grid, bool pair_box, hipStream_t s) {
  if (a.n_pairs <= 0) return hipSuccess;
  if (a.stats_on) hipLaunchKernelGGL(k_batch_clear_stats, dim3(1), dim3(kWave), 0, s, a.st);
  // the instances with counters run the same grids as those without (a
  // workgroup the device cannot hold yet waits its turn; no wave waits on
  // another)
  const dim3 b(kSweepWaves * kWave);
  if (pair_box && a.ring_tiles) {
    // few registers: as many workgroups as of the sweep are resident
    if (a.stats_on) {
      hipLaunchKernelGGL(k_ring_tiles<true>, dim3(sweep_grid), b, 0, s, a);
      hipLaunchKernelGGL(k_tile_pairs<true>, dim3(sweep_grid), b, 0, s, a);
    } else {
      hipLaunchKernelGGL(k_ring_tiles<false>, dim3(sweep_grid), b, 0, s, a);
      hipLaunchKernelGGL(k_tile_pairs<false>, dim3(sweep_grid), b, 0, s, a);
    }
  }
  if (pair_box && a.stats_on)
    hipLaunchKernelGGL((k_batch_sweep<true, true>), dim3(sweep_grid), b, 0, s, a);
  else if (pair_box)
    hipLaunchKernelGGL((k_batch_sweep<true, false>), dim3(sweep_grid), b, 0, s, a);
  else if (a.stats_on)
    hipLaunchKernelGGL((k_batch_sweep<false, true>), dim3(sweep_grid), b, 0, s, a);
  else
    hipLaunchKernelGGL((k_batch_sweep<false, false>), dim3(sweep_grid), b, 0, s, a);
  const dim3 bm(kTeamWaves * kWave);
  if (a.stats_on)
    hipLaunchKernelGGL(k_batch_medium<true>, dim3(medium_grid), bm, 0, s, a);
  else
    hipLaunchKernelGGL(k_batch_medium<false>, dim3(medium_grid), bm, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_batch_persistent(const BatchArgs& a, int grid, int waves_per_wg, hipStream_t s) {
  if (a.n_pairs <= 0) return hipSuccess;
  const size_t lds = (size_t)waves_per_wg * batch_lds_bytes_per_wave();
  if (a.stats_on)
    hipLaunchKernelGGL(k_batch_run<true>, dim3(grid), dim3(waves_per_wg * kWave), lds, s, a);
  else
    hipLaunchKernelGGL(k_batch_run<false>, dim3(grid), dim3(waves_per_wg * kWave), lds, s, a);
  return hipGetLastError();
}

}  // namespace sccg
