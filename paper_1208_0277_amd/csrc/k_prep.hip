// Per-polygon prepass, ring validation and the set-level Jaccard reduction.
#include <limits.h>

#include "fix192.h"
#include "sccg_device.h"

namespace sccg {

// A row of 16 lanes per ring, four rings per wave: lane j of the row takes
// vertices j, 16 + j, 32 + j and 48 + j of each 64, four loads in flight of
// 128 neighbouring bytes each; past the ring's end it takes the first vertex
// again, which leaves extents alone and is the last vertex's successor.  A
// vertex's successor comes from the next lane, lane 15's from lane 0 of the
// next 16.  Bound by the rings' bytes (one lane per ring read 8 bytes of 64
// lines at a time: 600,000 rings of 90 vertices validated in 850 us; eight
// lanes with the successors loaded again 147 us for extents and areas).
//
// Short rings leave most of a row idle.  Many of few vertices on average are
// taken 16 of a wave at a time, on the four lanes of a quad each, 16 vertices a
// step, whatever their own length.  The average is read on the device, and is
// where the two cross, on rows / on quads: a million rings validated, of 4
// vertices 55 / 27 us, 20 57 / 38, 32 62 / 48, 40 80 / 77, 48 83 / 85; extents and
// areas of two million, of 4 157 / 65 us, 20 160 / 87, 32 196 / 120, 48 236 / 199
// (a thread per ring validated the first in 28 us, eight lanes per ring took 64
// for the extents and areas of 4 vertices, 178 of 40).
constexpr int kRow = 16;        // lanes per ring (a DPP row)
constexpr int kRowChunks = 4;   // loads of a lane in flight
constexpr int kRowStep = kRow * kRowChunks;
constexpr int kRowRings = 256 / kRow;  // rings of a workgroup's rows
constexpr int kQuadStep = 4 * kRowChunks;
constexpr int kShortMeta = 48, kShortValidate = 32;  // vertices on average of rings taken on quads

struct RowChunk {
  int2 v[kRowChunks], s[kRowChunks];  // vertices and, where asked for, their successors
};
template <bool kSucc>
__device__ __forceinline__ RowChunk row_load(const int2* R, int64_t nv, int64_t base, int j) {
  RowChunk r;
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c) {
    const int64_t k = base + c * kRow + j;
    r.v[c] = R[k < nv ? k : 0];
  }
  if (kSucc) {
    const int2 nxt = R[base + kRowStep < nv ? base + kRowStep : 0];
#pragma unroll
    for (int c = 0; c < kRowChunks; ++c) {
      int2 t = nxt;  // lane 15's successor
      if (c + 1 < kRowChunks) {
        t.x = __builtin_amdgcn_update_dpp(0, r.v[c + 1 < kRowChunks ? c + 1 : c].x, 0x12f, 0xf, 0xf, false);  // row_ror:15
        t.y = __builtin_amdgcn_update_dpp(0, r.v[c + 1 < kRowChunks ? c + 1 : c].y, 0x12f, 0xf, 0xf, false);
      }
      r.s[c].x = __builtin_amdgcn_update_dpp(t.x, r.v[c].x, 0x101, 0xf, 0xf, false);  // row_shl:1
      r.s[c].y = __builtin_amdgcn_update_dpp(t.y, r.v[c].y, 0x101, 0xf, 0xf, false);
    }
  }
  return r;
}
// 16 vertices of a short ring on the four lanes of a quad (lane j of it).
template <bool kSucc>
__device__ __forceinline__ RowChunk quad_load(const int2* R, int64_t nv, int64_t base, int j) {
  RowChunk r;
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c) r.v[c] = R[base + c * 4 + j < nv ? base + c * 4 + j : 0];
  if (kSucc) {
    int2 next = R[base + kQuadStep < nv ? base + kQuadStep : 0];  // lane 3's successor in the last chunk
#pragma unroll
    for (int c = kRowChunks - 1; c >= 0; --c) {
      // quad_perm 1 2 3 0: the next lane's, and in lane 3 lane 0's
      const int2 t = make_int2(__builtin_amdgcn_update_dpp(0, r.v[c].x, 0x39, 0xf, 0xf, false),
                               __builtin_amdgcn_update_dpp(0, r.v[c].y, 0x39, 0xf, 0xf, false));
      r.s[c] = j == 3 ? next : t;
      next = t;
    }
  }
  return r;
}
__device__ __forceinline__ int32_t quad_min(int32_t x) {
  x = min(x, __builtin_amdgcn_update_dpp(x, x, 0xb1, 0xf, 0xf, false));
  return min(x, __builtin_amdgcn_update_dpp(x, x, 0x4e, 0xf, 0xf, false));
}

__device__ __forceinline__ int32_t row_min(int32_t x) {
  x = min(x, __builtin_amdgcn_update_dpp(x, x, 0xb1, 0xf, 0xf, false));
  x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x4e, 0xf, 0xf, false));
  x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x141, 0xf, 0xf, false));
  return min(x, __builtin_amdgcn_update_dpp(x, x, 0x140, 0xf, 0xf, false));
}
__device__ __forceinline__ uint32_t row_sum(uint32_t u) {
  int x = (int)u;
  x += __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, false);
  return (uint32_t)(x + __builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, false));
}

// A ring of one of two sets, by its number over both.
struct RingOf {
  bool second;
  int64_t k, nv;
  const int2* R;
  __device__ __forceinline__ RingOf(const Polys& A, const Polys& B, int64_t at) {
    second = at >= A.n;
    k = second ? at - A.n : at;
    const int64_t* off = second ? B.off : A.off;
    const int64_t o = off[k];
    nv = off[k + 1] - o;
    R = (second ? B.xy : A.xy) + o;
  }
};

// What a lane's vertices add to its ring's extent (minima, and complemented
// maxima) and doubled area.
struct RingAcc {
  int32_t x0 = INT_MAX, y0 = INT_MAX, nx1 = INT_MAX, ny1 = INT_MAX;
  uint32_t tn = 0;
  template <bool kArea>
  __device__ __forceinline__ void add(const RowChunk& r, int2 f) {
#pragma unroll
    for (int c = 0; c < kRowChunks; ++c) {
      x0 = min(x0, r.v[c].x);
      y0 = min(y0, r.v[c].y);
      nx1 = min(nx1, ~r.v[c].x);
      ny1 = min(ny1, ~r.v[c].y);
      if (kArea)
        tn += (uint32_t)__mul24((int)((uint32_t)r.v[c].x + (uint32_t)r.s[c].x - 2u * (uint32_t)f.x),
                                (int)((uint32_t)r.s[c].y - (uint32_t)r.v[c].y));
    }
  }
};
// twice the signed area modulo 2^64 of a lane's edges
__device__ __forceinline__ uint64_t wide_area(const RowChunk& r) {
  uint64_t t = 0;
  for (int c = 0; c < kRowChunks; ++c)
    t += (uint64_t)((int64_t)r.v[c].x * r.s[c].y) - (uint64_t)((int64_t)r.s[c].x * r.v[c].y);
  return t;
}
template <int kLanes>
__device__ __forceinline__ uint64_t lanes_sum64(uint64_t v) {
  for (int d = 1; d < kLanes; d <<= 1) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, d, kWave);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), d, kWave);
    v += ((uint64_t)hi << 32) | lo;
  }
  return v;
}
__device__ __forceinline__ int64_t half_size(int64_t t) { return (int64_t)((t < 0 ? 0 - (uint64_t)t : (uint64_t)t) / 2); }
// Whether twice a ring's signed area fits 32 bits and its terms 24: a ring of nv
// vertices runs at most nv / 2 times around any pixel of its extent.
__device__ __forceinline__ bool narrow(const Meta& m, int64_t nv) {
  const uint32_t w = side_u(m.x0, m.x1), h = side_u(m.y0, m.y1);
  return max(w, h) <= (uint32_t)kMaxSide && (uint64_t)nv * (w * h) < (uint64_t)1 << 31;
}

__device__ __forceinline__ bool beyond(const Meta& m) {
  return m.x0 < -kMaxCoord || m.y0 < -kMaxCoord || m.x1 > kMaxCoord || m.y1 > kMaxCoord;
}

// A ring's results, by its first lane.
template <bool kArea>
__device__ __forceinline__ void put_meta(const RingOf& g, const Meta& m, bool bad, int64_t area, Meta* metaA,
                                         int64_t* areaA, Meta* metaB, int64_t* areaB, uint32_t* err) {
  if (bad) latch_error(err, kErrCoord);
  Meta* to = g.second ? metaB : metaA;
  *reinterpret_cast<int4*>(to + g.k) =
      bad || g.nv <= 0 ? make_int4(INT_MAX, INT_MAX, INT_MIN, INT_MIN) : make_int4(m.x0, m.y0, m.x1, m.y1);
  int64_t* areas = g.second ? areaB : areaA;
  if (kArea) areas[g.k] = area;
}
// A ring on the 16 lanes of a row (lane j of it), `on` or an idle row.
template <bool kArea>
__device__ __forceinline__ void row_meta(const RingOf& g, bool on, int j, Meta* metaA, int64_t* areaA, Meta* metaB,
                                         int64_t* areaB, uint32_t* err) {
  const int64_t nv = on ? g.nv : 0;
  RingAcc acc;
  int2 f = make_int2(0, 0);
  if (kArea && nv > 0) f = g.R[0];
  for (int64_t base = 0; base < nv; base += kRowStep) acc.add<kArea>(row_load<kArea>(g.R, nv, base, j), f);
  const Meta m{row_min(acc.x0), row_min(acc.y0), ~row_min(acc.nx1), ~row_min(acc.ny1)};
  const bool bad = nv > 0 && beyond(m);
  int64_t area = 0;
  if (kArea && nv > 0 && !bad) {
    if (narrow(m, nv)) {
      area = half_size((int32_t)row_sum(acc.tn));
    } else {
      uint64_t tw = 0;
      for (int64_t base = 0; base < nv; base += kRowStep) tw += wide_area(row_load<true>(g.R, nv, base, j));
      area = half_size((int64_t)lanes_sum64<kRow>(tw));
    }
  }
  if (j == 0 && on) put_meta<kArea>(g, m, bad, area, metaA, areaA, metaB, areaB, err);
}
// A short ring on the four lanes of a quad.
template <bool kArea>
__device__ __forceinline__ void quad_meta(const RingOf& g, bool on, int j, Meta* metaA, int64_t* areaA, Meta* metaB,
                                          int64_t* areaB, uint32_t* err) {
  const int64_t nv = on ? g.nv : 0;
  RingAcc acc;
  int2 f = make_int2(0, 0);
  if (kArea && nv > 0) f = g.R[0];
  for (int64_t base = 0; base < nv; base += kQuadStep) acc.add<kArea>(quad_load<kArea>(g.R, nv, base, j), f);
  const Meta m{quad_min(acc.x0), quad_min(acc.y0), ~quad_min(acc.nx1), ~quad_min(acc.ny1)};
  const bool bad = nv > 0 && beyond(m);
  int64_t area = 0;
  if (kArea && nv > 0 && !bad) {
    if (narrow(m, nv)) {
      int t = (int)acc.tn;
      t += __builtin_amdgcn_update_dpp(0, t, 0xb1, 0xf, 0xf, false);
      t += __builtin_amdgcn_update_dpp(0, t, 0x4e, 0xf, 0xf, false);
      area = half_size(t);
    } else {
      uint64_t tw = 0;
      for (int64_t base = 0; base < nv; base += kQuadStep) tw += wide_area(quad_load<true>(g.R, nv, base, j));
      area = half_size((int64_t)lanes_sum64<4>(tw));
    }
  }
  if (j == 0 && on) put_meta<kArea>(g, m, bad, area, metaA, areaA, metaB, areaB, err);
}

// Rings with few vertices on average: the workgroups below `quads` take 64 of a
// wave at a time, 16 at once on the four lanes of a quad each, and the others
// none.  f(ring, on) is called by the quads.
__device__ __forceinline__ bool mostly_short(int64_t verts, int64_t rings, int most) { return verts <= most * rings; }
template <typename F>
__device__ __forceinline__ void on_quads(const Polys& A, const Polys& B, unsigned quads, F f) {
  const int64_t n = A.n + B.n;
  if (blockIdx.x >= quads) return;
  for (int64_t k0 = uniform64((int64_t)blockIdx.x * 256 + threadIdx.x / kWave * kWave); k0 < n;
       k0 = uniform64(k0 + (int64_t)quads * 256))
#pragma unroll 1
    for (int i = 0; i < kWave && k0 + i < n; i += kWave / 4) {
      const int64_t at = k0 + i + lane_id() / 4;
      f(RingOf(A, B, min(at, n - 1)), at < n);
    }
}
// Where a launch looks at the average at all (fewer rings take as long in rows).
unsigned quad_blocks(int64_t n) { return n >= int64_t(1) << 17 ? blocks_of(n, 256) : 0u; }

// Extents, and kArea |shoelace|/2 (Section 3.2's area formula), of the rings
// of one or two sets.  Twice the signed area is summed as (x + x') (y' - y)
// over the edges, x relative to the first vertex, modulo 2^32 where that holds
// it (see narrow); else again modulo 2^64, in which it (at most 2^63 in size)
// is exact.
template <bool kArea>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8)))
k_meta_rows(Polys A, Meta* metaA, int64_t* areaA, Polys B, Meta* metaB, int64_t* areaB, uint32_t* err, unsigned quads) {
  const int64_t n = A.n + B.n;
  if (quads && mostly_short(A.off[A.n] + B.off[B.n], n, kShortMeta)) {
    on_quads(A, B, quads, [&](const RingOf& g, bool on) {
      quad_meta<kArea>(g, on, lane_id() & 3, metaA, areaA, metaB, areaB, err);
    });
    return;
  }
  for (int64_t k0 = (int64_t)blockIdx.x * kRowRings; k0 < n; k0 += (int64_t)gridDim.x * kRowRings) {
    const int64_t at = k0 + threadIdx.x / kRow;
    if (at < n) row_meta<kArea>(RingOf(A, B, at), true, threadIdx.x % kRow, metaA, areaA, metaB, areaB, err);
  }
}

template <bool kArea>
void launch_meta(const Polys& A, Meta* metaA, int64_t* areaA, const Polys& B, Meta* metaB, int64_t* areaB, uint32_t* err,
                 hipStream_t s) {
  const int64_t n = A.n + B.n;
  hipLaunchKernelGGL(k_meta_rows<kArea>, dim3(blocks_of(n, kRowRings)), dim3(256), 0, s, A, metaA, areaA, B, metaB, areaB,
                     err, quad_blocks(n));
}
hipError_t launch_poly_meta(const Polys& A, Meta* metaA, int64_t* areaA, const Polys& B, Meta* metaB, int64_t* areaB,
                            uint32_t* err, hipStream_t s) {
  if (A.n + B.n <= 0) return hipSuccess;
  if (areaA)
    launch_meta<true>(A, metaA, areaA, B, metaB, areaB, err, s);
  else
    launch_meta<false>(A, metaA, areaA, B, metaB, areaB, err, s);
  return hipGetLastError();
}

// ---------------------------------------------------------------- validation
// -1 as the largest unsigned value: what the smallest bad index is taken from,
// and what is left when there is none
__global__ void k_validate_init(unsigned long long* first_bad) { *first_bad = ~0ull; }

// the smallest bad ring of a wave's lanes, whose rings k stand in order
__device__ __forceinline__ void report_bad(bool bad, int64_t k, unsigned long long* first_bad) {
  const uint64_t m = ballot(bad);
  if (m && lane_id() == __ffsll((long long)m) - 1 &&
      (unsigned long long)k < __hip_atomic_load(first_bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMin(first_bad, (unsigned long long)k);
}
__device__ __forceinline__ bool slanted(const RowChunk& r) {
  bool bad = false;
#pragma unroll
  for (int c = 0; c < kRowChunks; ++c) bad |= (r.v[c].x != r.s[c].x) & (r.v[c].y != r.s[c].y);
  return bad;
}
__global__ void __launch_bounds__(256) k_validate(Polys P, unsigned long long* first_bad, unsigned quads) {
  if (quads && mostly_short(P.off[P.n], P.n, kShortValidate)) {
    on_quads(P, Polys{}, quads, [&](const RingOf& g, bool on) {
      bool bad = g.nv < 4;
      for (int64_t base = 0; base < g.nv; base += kQuadStep) bad |= slanted(quad_load<true>(g.R, g.nv, base, lane_id() & 3));
      report_bad(on && bad, g.k, first_bad);
    });
    return;
  }
  for (int64_t k0 = (int64_t)blockIdx.x * kRowRings; k0 < P.n; k0 += (int64_t)gridDim.x * kRowRings) {
    const int64_t k = k0 + threadIdx.x / kRow;
    bool bad = false;
    if (k < P.n) {
      const int64_t o = P.off[k], nv = P.off[k + 1] - o;
      bad = nv < 4;
      for (int64_t base = 0; base < nv; base += kRowStep) bad |= slanted(row_load<true>(P.xy + o, nv, base, threadIdx.x % kRow));
    }
    report_bad(bad, k, first_bad);
  }
}

hipError_t launch_validate(const Polys& P, int64_t* first_bad, hipStream_t s) {
  auto* fb = reinterpret_cast<unsigned long long*>(first_bad);
  hipLaunchKernelGGL(k_validate_init, dim3(1), dim3(1), 0, s, fb);
  if (P.n > 0)
    hipLaunchKernelGGL(k_validate, dim3(blocks_of(P.n, kRowRings)), dim3(256), 0, s, P, fb, quad_blocks(P.n));
  return hipGetLastError();
}

// ------------------------------------------------------------------- Jaccard
// Per-set sums of Eq. 1 over the pairs of each set; J' by the exact ratio
// sum of fix192.h.  Every wave takes an equal range of consecutive pairs of the
// whole pair range, whatever sets they belong to, and adds up the pairs of one
// set after the other: integer sums, and the Fix192 ratio sum as six 32-bit
// limbs, each in a 64-bit sum of its own (at most 2^31 of them).  A set that
// lies within the range is finished there; of the set that the range starts
// in and the one it ends in the sums are left for a second pass over the sets
// that more than one wave has pairs of.  Integer and fixed-point addition do
// not depend on order, so the result is the same bits as any sequential sum.
// (Chunks claimed by workgroups, reduced in LDS and added with atomics: 83 us
// for 9.5M pairs of 64 sets.)
constexpr int kJacWords = 9;   // ratio sum limbs, then sums of I and U, and pairs
constexpr int kJacStep = 256;  // pairs that a wave takes at least
constexpr int kJacAhead = 4;   // pairs of a lane in flight
struct JacSums {
  uint64_t w[kJacWords];
};

// a wave's range of the pairs [base, end)
struct JacRange {
  int64_t per, base, end;
  __device__ __forceinline__ JacRange(int64_t n_sets, const int64_t* set_off, int64_t waves) {
    base = set_off[0];
    end = set_off[n_sets];
    per = max((int64_t)kJacStep, (end - base + waves - 1) / waves);
  }
  __device__ __forceinline__ int64_t wave_of(int64_t k) const { return (k - base) / per; }
};

__device__ __forceinline__ void jac_store(int64_t s, const JacSums& t, bool want_jp, int64_t* sum_i, int64_t* sum_u,
                                          int64_t* n_contrib, double* jout, double* jprime) {
  const int64_t tI = (int64_t)t.w[6], tU = (int64_t)t.w[7], tn = (int64_t)t.w[8];
  sum_i[s] = tI;
  sum_u[s] = tU;
  n_contrib[s] = tn;
  jout[s] = tU > 0 ? (double)tI / (double)tU : 0.0;
  if (want_jp) {
    // limb k weighs 2^(32 k): add them up with carries into three words
    Fix192 f;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      Fix192 x;
      const int w = k >> 1, off = 32 * (k & 1);
      x.w[w] = t.w[k] << off;
      if (off && w + 1 < 3) x.w[w + 1 < 3 ? w + 1 : w] = t.w[k] >> (64 - off);
      f.add(x);
    }
    jprime[s] = tn > 0 ? f.to_double() / (double)tn : 0.0;
  }
}

__global__ void __launch_bounds__(256) k_jaccard_waves(int64_t n_sets, const int64_t* set_off, const int64_t* inter,
                                                       const int64_t* uni, uint32_t flags, int64_t* sum_i,
                                                       int64_t* sum_u, int64_t* n_contrib, double* jout, double* jprime,
                                                       JacSums* part) {
  const bool include_zero = (flags & SCCG_J_INCLUDE_ZERO) != 0, want_jp = jprime != nullptr;
  const int lane = lane_id();
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
  const int64_t w = uniform64((int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
  const JacRange range(n_sets, set_off, waves);
  const int64_t r0 = uniform64(range.base + w * range.per), r1 = min(uniform64(r0 + range.per), uniform64(range.end));
  if (r0 >= r1) return;
  // the set holding pair r0: the last s with set_off[s] <= r0
  int64_t lo = 0, hi = n_sets;
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + kWave - 1) / kWave;
    const uint64_t m = ballot(lo + lane * step < hi && set_off[min(lo + lane * step, hi - 1)] <= r0);
    lo = uniform64(lo + (__popcll(m) - 1) * step);
    hi = uniform64(min(hi, lo + step));
  }
  int64_t o1 = r0;
  for (int64_t s = lo; o1 < r1; ++s) {
    const int64_t o0 = o1, set_end = uniform64(set_off[s + 1]);
    o1 = min(set_end, r1);
    if (o1 <= o0) continue;  // an empty set
    uint64_t si = 0, su = 0;
    uint32_t nn = 0;
    Fix192 fx;
    auto add = [&](int64_t I, int64_t U) {
      if (!include_zero && I == 0) return;
      si += (uint64_t)I;
      su += (uint64_t)U;
      nn += 1;
      if (want_jp && U > 0) fx.add_ratio((double)I / (double)U);
    };
    int64_t k = o0 + lane;
    for (; k + (kJacAhead - 1) * kWave < o1; k += kJacAhead * kWave) {
      int64_t I[kJacAhead], U[kJacAhead];
#pragma unroll
      for (int u = 0; u < kJacAhead; ++u) {
        I[u] = inter[k + u * kWave];
        U[u] = uni[k + u * kWave];
      }
#pragma unroll
      for (int u = 0; u < kJacAhead; ++u) add(I[u], U[u]);
    }
    for (; k < o1; k += kWave) add(inter[k], uni[k]);
    JacSums t;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      t.w[2 * k] = want_jp ? wave_sum_u64(fx.w[k] & 0xffffffffull) : 0ull;
      t.w[2 * k + 1] = want_jp ? wave_sum_u64(fx.w[k] >> 32) : 0ull;
    }
    t.w[6] = wave_sum_u64(si);
    t.w[7] = wave_sum_u64(su);
    t.w[8] = wave_sum_u32(nn);
    const bool from = o0 == r0 && uniform64(set_off[s]) < r0, on = set_end > r1;
    if (lane == 0) {
      if (!from && !on)
        jac_store(s, t, want_jp, sum_i, sum_u, n_contrib, jout, jprime);
      else
        part[2 * w + (from ? 0 : 1)] = t;  // a set begun before, or first met here
    }
  }
}

// The sets that no wave finished: empty ones, and those with pairs of several
// waves, whose sums the waves left.  kWaves waves per set: a workgroup for
// each of few sets, which may have thousands of sums each, else one wave.
template <int kWaves>
__global__ void __launch_bounds__(256) k_jaccard_sets(int64_t n_sets, const int64_t* set_off, int64_t waves,
                                                      const JacSums* part, int64_t* sum_i, int64_t* sum_u,
                                                      int64_t* n_contrib, double* jout, double* jprime, int64_t first) {
  __shared__ JacSums sh[4];
  const int lane = lane_id(), me = (int)(threadIdx.x / kWave) % kWaves;
  const int64_t s = first + ((int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave) / kWaves;
  if (s >= n_sets) return;
  const JacRange range(n_sets, set_off, waves);
  const int64_t o0 = set_off[s], o1 = set_off[s + 1];
  JacSums t{};
  if (o0 < o1) {
    const int64_t w0 = range.wave_of(o0), w1 = range.wave_of(o1 - 1);
    if (w0 == w1) return;
    uint64_t x[kJacWords] = {};
    for (int64_t w = w0 + me * kWave + lane; w <= w1; w += kWaves * kWave) {
      const JacSums& p = part[2 * w + (w == w0 ? 1 : 0)];
#pragma unroll
      for (int k = 0; k < kJacWords; ++k) x[k] += p.w[k];
    }
#pragma unroll
    for (int k = 0; k < kJacWords; ++k) t.w[k] = wave_sum_u64(x[k]);
  }
  if (kWaves > 1) {
    if (lane == 0) sh[me] = t;
    __syncthreads();
    if (me == 0)
      for (int u = 1; u < kWaves; ++u)
#pragma unroll
        for (int k = 0; k < kJacWords; ++k) t.w[k] += sh[u].w[k];
  }
  if (lane == 0 && me == 0) jac_store(s, t, jprime != nullptr, sum_i, sum_u, n_contrib, jout, jprime);
}

int64_t jaccard_scratch(int waves) { return 2 * (int64_t)waves * (int64_t)sizeof(JacSums); }

hipError_t launch_jaccard(int64_t n_sets, const int64_t* set_off, const int64_t* inter, const int64_t* uni,
                          uint32_t flags, int64_t* sum_i, int64_t* sum_u, int64_t* n_contrib, double* j,
                          double* jprime, void* scratch, int waves, hipStream_t s) {
  if (n_sets <= 0) return hipSuccess;
  JacSums* part = static_cast<JacSums*>(scratch);
  hipLaunchKernelGGL(k_jaccard_waves, dim3((unsigned)waves / 4), dim3(256), 0, s, n_sets, set_off, inter, uni, flags,
                     sum_i, sum_u, n_contrib, j, jprime, part);
  if (n_sets <= 2048)
    hipLaunchKernelGGL(k_jaccard_sets<4>, dim3((unsigned)n_sets), dim3(256), 0, s, n_sets, set_off, (int64_t)waves, part,
                       sum_i, sum_u, n_contrib, j, jprime, 0);
  else
    for_slices(n_sets, 256 / kWave, [&](int64_t first, unsigned blocks) {
      hipLaunchKernelGGL(k_jaccard_sets<1>, dim3(blocks), dim3(256), 0, s, n_sets, set_off, (int64_t)waves, part, sum_i,
                         sum_u, n_contrib, j, jprime, first);
    });
  return hipGetLastError();
}

}  // namespace sccg
