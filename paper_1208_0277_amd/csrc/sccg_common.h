// Internal declarations shared by the device library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sccg.h"

namespace sccg {

constexpr int kWave = 64;
constexpr int32_t kMaxSide = 32767;        // largest accepted pair-box side (pixels)
constexpr int32_t kMaxCoord = 1 << 30;     // largest accepted |coordinate|
constexpr int kTile = 64;                  // leaf tile side of the batched path (pixels)
constexpr int kMaxGrid = 8;                // batched split grid is at most 8 x 8 cells

// Device error word bits (latched, reported by sccg_sync).
enum : uint32_t {
  kErrIndex = 1u,     // pair index outside its polygon set
  kErrSide = 2u,      // pair-box side above kMaxSide
  kErrCoord = 4u,     // |coordinate| above kMaxCoord
  kErrWatchdog = 8u,  // a bounded wait in the persistent kernel ran out
};

// Classes of a pair by its box: nothing to count, one leaf tile, or larger.
enum : uint8_t { kClsDone = 0, kClsSmall = 1, kClsLarge = 2 };

struct Polys {
  int64_t n;
  const int64_t* off;
  const int2* xy;
};

// Vertex extent of a polygon: pixels [x0,x1) x [y0,y1).  x0 > x1 marks an
// empty or rejected polygon.
struct Meta {
  int32_t x0, y0, x1, y1;
};

// Number of statistics counters (see sccg_get_stats).
constexpr int kNumStats = 16;

// Workgroups of a kernel that takes `n` items, `per` each.  A dispatch has fewer
// than 2^32 threads: of a kernel with several lanes per item a grid stops at
// 2^20 workgroups, and the kernel goes over it again, or is launched again from
// the item it got to (the loop cost the join's writing pass 33.9 -> 38.6 us, a
// first item 35.1; the per-ring passes were no slower with it).
constexpr int64_t kMostBlocks = int64_t(1) << 20;
constexpr unsigned blocks_of(int64_t n, int64_t per) {
  const int64_t b = (n + per - 1) / per;
  return (unsigned)(b < 1 ? 1 : b < kMostBlocks ? b : kMostBlocks);
}
// launch(first item, workgroups), at least once
template <typename F>
void for_slices(int64_t n, int64_t per, F launch) {
  int64_t first = 0;
  do {
    launch(first, blocks_of(n - first, per));
    first += kMostBlocks * per;
  } while (first < n);
}

// ------------------------------------------------------------------ launches
// Each returns a hipError_t from the launch.

// Per polygon of A and B: vertex extent, coordinate range check, and, unless
// the area arrays are NULL, |shoelace|/2.
hipError_t launch_poly_meta(const Polys& A, Meta* metaA, int64_t* areaA, const Polys& B, Meta* metaB, int64_t* areaB,
                            uint32_t* err, hipStream_t s);

struct PlainArgs {
  Polys A, B;
  const Meta* metaA;
  const Meta* metaB;
  const int64_t* areaA;
  const int64_t* areaB;
  int64_t n_pairs;
  const int32_t* pa;
  const int32_t* pb;
  int64_t* inter;
  int64_t* uni;
  uint32_t* err;
  unsigned long long* stats;  // nullable
  int32_t box_threshold;
  int32_t gx, gy;
  int32_t lds_vertex_cap;
};
hipError_t launch_plain(const PlainArgs& a, int wg_size, int grid, hipStream_t s);
int plain_lds_bytes(int wg_size, int lds_vertex_cap);
int plain_occupancy(int wg_size, int lds_vertex_cap);

// A device counter on a cache line of its own, so that claims on different
// counters never contend for one line.
struct alignas(128) Counter {
  unsigned long long v;
  unsigned long long pad[15];
};

// Work is claimed from kStreams interleaved streams (one per XCD): stream s
// owns entries s, s + kStreams, s + 2 kStreams, ... of a list.
constexpr int kStreams = 8;

// Device-side state of the batched path (one block of device memory), zero
// before the first call; the kernels of each call leave it ready for the next.
// Listed pairs are kept in kLptBuckets lists by vertex count (the cost the
// sweep can see): at least 4, 2 or 1 times heavy_verts, and the rest;
// the persistent kernel claims the largest bucket first.
constexpr int kLptBuckets = 4;
// How a kernel shares n items out among its waves: runs of consecutive items
// (at most `longest`), dealt out in turns.  A wave's whole share is at least
// 32 runs where there are that many items, so that shares differ by little.
constexpr int64_t share_run(int64_t n, int64_t waves, int64_t longest) {
  const int64_t r = n / (waves * 32);
  return r < 1 ? 1 : (r < longest ? r : longest);
}
// the largest share
constexpr int64_t most_share(int64_t n, int64_t waves, int64_t longest) {
  const int64_t run = share_run(n, waves, longest), full = n / (waves * run), rest = n - full * waves * run;
  return full * run + (rest < run ? rest : run);
}

// The most pairs that the workgroups of one stream of the union sweep take
// (`grid` workgroups of `per_wg` waves, shares of at most `most` pairs), and
// room for it whatever the grid, of up to 6000 workgroups: shares differ by at
// most a 32nd and one pair.
constexpr int64_t stream_cap_of(int64_t grid, int64_t per_wg, int64_t most) {
  return (grid + kStreams - 1) / kStreams * per_wg * most;
}
constexpr int64_t stream_cap_room(int64_t n_pairs) { return (n_pairs + n_pairs / 16) / kStreams + 3072; }
// The most pairs that the workgroups of one stream of the medium sweep (`grid`
// of them) list for the persistent kernel: every eighth long pair and their
// shares of the medium ones; and room for it whatever the grid, of 32 to 6000
// workgroups.
constexpr int64_t run_cap_of(int64_t n_pairs, int64_t grid) { return n_pairs / kStreams + grid / 4 + n_pairs / grid + 16; }
constexpr int64_t run_cap_room(int64_t n_pairs) { return n_pairs / kStreams + n_pairs / 32 + 2048; }
// 4-byte list entries for n pairs: the sweep's lists (long buckets, medium),
// the persistent kernel's buckets
constexpr int64_t pair_list_room(int64_t n) {
  return (kLptBuckets + 1) * kStreams * stream_cap_room(n) + kLptBuckets * kStreams * run_cap_room(n);
}

// Those of all buckets on one line: every wave of the persistent kernel reads
// them (32 lines each cost a call of 20,000 pairs 0.3 us).
struct alignas(128) BucketCounters {
  unsigned long long v[kLptBuckets];
};

struct BatchState {
  BucketCounters l_count[kStreams];  // pairs listed for the persistent kernel per stream and bucket
  Counter l_next[kStreams];      // per-stream claim counters over them, one after the other
  Counter m_count[kStreams];  // medium pairs listed by the sweep per stream
  Counter p_count[kLptBuckets][kStreams];  // long pairs listed by the sweep per bucket and stream
  Counter p_next[kStreams];      // per-stream claim counters over the long pairs
  Counter t_count[kStreams];  // pairs that the rings' tiles left per stream (cleared by the call that uses it)
  Counter q_head[kMaxGrid];   // per-queue ticket counters
  Counter q_tail[kMaxGrid];   // per-queue reservation counters
  unsigned long long stats[kNumStats];
};

struct BatchArgs {
  Polys A, B;
  int64_t n_pairs;
  const int32_t* pa;
  const int32_t* pb;
  int64_t* inter;
  int64_t* uni;
  uint32_t* err;
  uint8_t* cls;                  // [n_pairs] class of a pair listed for the persistent kernel
  // The sweep's lists: every stream has a part of its own, stream_cap entries
  // long, which the workgroups blockIdx % kStreams append to
  int32_t* l_list;               // [kLptBuckets][kStreams][stream_cap] long pairs
  int32_t* m_list;               // [kStreams][stream_cap] medium pairs
  int64_t stream_cap;            // see stream_cap_of
  int32_t* run_list;             // [kLptBuckets][kStreams][run_cap] pairs listed for the persistent kernel
  int32_t run_cap;               // see run_cap_of
  Meta* hbox;                    // [n_pairs] pair box of a listed pair (by pair index)
  BatchState* st;
  unsigned long long* queue;     // [n_queues * queue_cap] task words, 0 = empty
  int32_t queue_cap;             // slots per queue
  int32_t n_queues;
  int32_t chunk;                 // small pairs per claim
  int32_t heavy_verts;           // pairs with at least this many vertices are claimed first
  int32_t min_cells_to_queue;    // a split pushes its boxes to the queue only from this many boxes
  int32_t min_classify_cells;    // a leaf-level split classifies its tiles only from this many cells
  uint32_t flags;                // SCCG_F_*
  int32_t stats_on;
  // The rings' tiles (null: the call has none), A's rings, then B's: a ring's
  // columns from its leftmost on, one 64-bit mask of rows each, the lowest row
  // first; its box; and its pixels (with the vertices above bit 16; 0 of a
  // ring that no tile holds) and its area.
  uint64_t* ring_tiles;          // [rings][kTile], and one column
  Meta* ring_box;
  uint2* ring_sums;
  // nullable: per wave, (start, end) stamps of the device's constant-rate
  // counter, wave_cap waves per kernel: the sweep, the medium sweep, then
  // the persistent kernel
  unsigned long long* wave_t;
  int32_t wave_cap;
};
// kernels whose waves are stamped (see BatchArgs::wave_t)
constexpr int kStampedKernels = 3;
// The union sweep (sweep_grid workgroups; with ring_tiles, after the kernels
// that make and use them), then the medium sweep with the long pairs
// (medium_grid); pair_box: the union sweep also counts the pairs whose pair box
// fits a leaf tile (else the medium sweep does).
hipError_t launch_batch_sweeps(const BatchArgs& a, int sweep_grid, int medium_grid, bool pair_box, hipStream_t s);
// Whether a call of the union sweep with pair boxes pixelizes every ring once
// beforehand.  Making a ring's tile takes about what using it for a pair saves,
// and the two launches what they save for some 50,000 (dense tiles, the sweep
// alone against this: 2.69M pairs of 1.22M rings 1025 -> 640 us, 1.34M
// 579 -> 537, 896,000 424 -> 502; 168,000 of 76,000 108 -> 73, 84,000 64 -> 68;
// 41,000 of 19,000 41 -> 51; 9.5M of 4.8M with their set sums 3.50 -> 2.21 ms).
// Where hardly a ring fits a tile the two passes are lost: the 331,000 pairs of
// 151,000 rings of dense tiles scaled by 1 188 -> 100 us, by 2 366 -> 417, by 4
// 513 -> 560 (the rings' sizes are not known before they are read).  Offsets of
// tiles are 32 bits.
constexpr int64_t kRingTilesMost = (int64_t(1) << 23) - 1;  // 4.5 GB of scratch
constexpr int64_t kRingTilePairs = 49152;
constexpr bool use_ring_tiles(int64_t rings, int64_t n_pairs) {
  return rings <= kRingTilesMost && n_pairs >= rings + kRingTilePairs;
}
constexpr int64_t ring_tiles_bytes(int64_t rings) {
  return rings * (int64_t)(kTile * sizeof(uint64_t) + sizeof(Meta) + sizeof(uint2)) + 64;
}
// The persistent kernel (grid workgroups).
hipError_t launch_batch_persistent(const BatchArgs& a, int grid, int waves_per_wg, hipStream_t s);
int batch_lds_bytes_per_wave();
int batch_occupancy(int waves_per_wg);
// Workgroups per CU of the union sweep (the instance that counts pair boxes
// or the one that does not) and of the medium sweep.
int batch_sweep_occupancy(bool pair_box);
int batch_medium_occupancy();
int batch_sweep_waves_per_wg();
int batch_medium_waves_per_wg();

// Set-level Jaccard on `waves` waves (a multiple of 4), with jaccard_scratch
// bytes of scratch.
int64_t jaccard_scratch(int waves);
hipError_t launch_jaccard(int64_t n_sets, const int64_t* set_off, const int64_t* inter, const int64_t* uni,
                          uint32_t flags, int64_t* sum_i, int64_t* sum_u, int64_t* n_contrib, double* j,
                          double* jprime, void* scratch, int waves, hipStream_t s);

// Ring validation.
hipError_t launch_validate(const Polys& P, int64_t* first_bad, hipStream_t s);

// Filter stage (candidate pairs by MBR intersection): one call's arrays and
// the room in them.  `count` is all zero before and, when everything fitted,
// after.
int64_t scan_scratch(int64_t n);
int64_t join_found_room(int64_t n_b);
struct JoinLaunch {
  Polys A, B;
  const Meta* metaA;
  const Meta* metaB;
  int64_t n_sets;
  const int64_t* a_off;
  const int64_t* b_off;
  int cell;
  int4* bbox;            // [n_sets]
  int4* grid;            // [n_sets]
  int64_t* cell_base;    // [n_sets + 1]
  int64_t cell_room;     // cells that count and start hold
  int32_t* count;        // [cell_room]
  int64_t* start;        // [cell_room + 1]
  int64_t list_room;
  int32_t* list;         // [list_room]
  int64_t* sums;         // [scan_scratch of the most of cell_room, B.n and n_sets]
  int32_t* b_count;      // [B.n]
  int64_t* b_start;      // [B.n + 1]
  int32_t* found;        // [join_found_room(B.n)]
  int64_t cap;
  int32_t* out_pa;
  int32_t* out_pb;
  int64_t* out_set_off;
  int64_t* sizes;        // [3]: cells, entries (0 when the cells did not fit), pairs (0 when either did not)
  uint32_t* err;
};
hipError_t launch_join(const JoinLaunch& l, hipStream_t s);

// Section 3.4's operators from counts and edges.
hipError_t launch_relate(const Polys& A, const Polys& B, const Meta* metaA, const Meta* metaB, const int64_t* areaA,
                         const int64_t* areaB, int64_t n_pairs, const int32_t* pa, const int32_t* pb,
                         const int64_t* inter, uint32_t* out, uint32_t* err, hipStream_t s);

// Diagnostics: 32 integer VALU operations per lane and loop trip, `iters`
// trips, grid workgroups of 256 lanes.
hipError_t launch_valu_peak(int grid, int iters, unsigned long long* sink, hipStream_t s);

// The device error word of a context (read and cleared by the server, which
// owns its context and runs on the context's stream).
uint32_t* ctx_error_word(sccg_ctx* c);
// The context's calls make no ring tiles: of the server's arena only the rings
// that the pairs name are there, the other slots hold anything and are written
// while a call runs.
void ctx_without_ring_tiles(sccg_ctx* c);

}  // namespace sccg
