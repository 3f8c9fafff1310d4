// Section 3.4's other operators from the same machinery: containment and
// equality from the intersection count and the polygon areas, and touching
// (no common pixel, boundaries that share a point) from the edges.
//
// A lane per pair settles the pairs with a common pixel and those whose closed
// MBRs do not meet.  The others take the wave, one after the other: only edges
// that touch the common part of the two MBRs can meet an edge of the other
// ring, and of objects without a common pixel those are few; each of q's is
// tested against 64 of p's at a time.  (A wave per pair that walked all of q's
// edges one load after the other: 451,000 candidate pairs of dense tiles, a
// third of them without a common pixel, 2116 us.)
#include <limits.h>

#include "sccg_device.h"

namespace sccg {

namespace {

// The bounding box of an edge; an axis-parallel edge, as a closed segment, is
// its own box.
struct EdgeBox {
  int x0, y0, x1, y1;
};
__device__ __forceinline__ EdgeBox edge_box(int2 v, int2 w) {
  return EdgeBox{min(v.x, w.x), min(v.y, w.y), max(v.x, w.x), max(v.y, w.y)};
}
__device__ __forceinline__ bool boxes_meet(const EdgeBox& a, const EdgeBox& b) {
  return (max(a.x0, b.x0) <= min(a.x1, b.x1)) & (max(a.y0, b.y0) <= min(a.y1, b.y1));
}
__device__ __forceinline__ EdgeBox lane_box(const EdgeBox& e, int l) {
  return EdgeBox{__builtin_amdgcn_readlane(e.x0, l), __builtin_amdgcn_readlane(e.y0, l),
                 __builtin_amdgcn_readlane(e.x1, l), __builtin_amdgcn_readlane(e.y1, l)};
}
// The lane's edge of a ring's chunk from `base`, and the lanes that have one
// touching `in`.
__device__ __forceinline__ uint64_t chunk_edges(const int2* R, int64_t n, int64_t base, int lane, const EdgeBox& in,
                                                EdgeBox& e) {
  const int64_t i = min(base + lane, n - 1);
  e = edge_box(R[i], R[i + 1 == n ? 0 : i + 1]);
  return ballot((base + lane < n) & boxes_meet(e, in));
}

}  // namespace

// `per` pairs per wave (a power of two up to 64: fewer when there are few
// pairs, so that more waves share the pairs that take a whole one).
__global__ void __launch_bounds__(256) k_relate(Polys A, Polys B, const Meta* metaA, const Meta* metaB,
                                                const int64_t* areaA, const int64_t* areaB, int64_t n_pairs,
                                                const int32_t* pa, const int32_t* pb, const int64_t* inter,
                                                uint32_t* out, uint32_t* err, int per, int64_t first) {
  const int lane = lane_id();
  const int64_t k = first + ((int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave) * per + lane;
  const bool live = lane < per && k < n_pairs;
  uint32_t r = 0;
  bool near = false;
  EdgeBox common{0, 0, 0, 0};
  int64_t op = 0, oq = 0;
  int np = 0, nq = 0;
  if (live) {
    const int64_t a = pa[k], b = pb[k];
    if (a < 0 || a >= A.n || b < 0 || b >= B.n) {
      latch_error(err, kErrIndex);
    } else {
      const int64_t I = inter[k];
      if (I > 0) {
        const int64_t ap = areaA[a], aq = areaB[b];
        r |= SCCG_REL_INTERSECTS;
        if (I == aq) r |= SCCG_REL_CONTAINS;
        if (I == ap) r |= SCCG_REL_WITHIN;
        if (I == ap && I == aq) r |= SCCG_REL_EQUALS;
      } else {
        // MBR extents are [x0, x1) in pixels: the vertices span [x0, x1] x [y0, y1]
        const Meta mp = load_meta(metaA, a), mq = load_meta(metaB, b);
        common = EdgeBox{max(mp.x0, mq.x0), max(mp.y0, mq.y0), min(mp.x1, mq.x1), min(mp.y1, mq.y1)};
        near = mp.x0 < mp.x1 && mq.x0 < mq.x1 && common.x0 <= common.x1 && common.y0 <= common.y1;
        if (near) {
          op = A.off[a];
          np = (int)(A.off[a + 1] - op);
          oq = B.off[b];
          nq = (int)(B.off[b + 1] - oq);
        }
      }
    }
  }
  uint64_t todo = ballot(near), touching = 0;
  while (todo) {
    const int l = __ffsll((long long)todo) - 1;
    todo &= todo - 1;
    const EdgeBox in = lane_box(common, l);
    const int n_p = __builtin_amdgcn_readlane(np, l), n_q = __builtin_amdgcn_readlane(nq, l);
    const int2* P = A.xy + uniform64(__shfl((long long)op, l, kWave));
    const int2* Q = B.xy + uniform64(__shfl((long long)oq, l, kWave));
    uint64_t met = 0;
    for (int bp = 0; bp < n_p && !met; bp += kWave) {
      EdgeBox ep, eq;
      const uint64_t mp = chunk_edges(P, n_p, bp, lane, in, ep);
      if (!mp) continue;
      for (int bq = 0; bq < n_q && !met; bq += kWave) {
        uint64_t mq = chunk_edges(Q, n_q, bq, lane, in, eq);
        while (mq && !met) {
          const EdgeBox one = lane_box(eq, __ffsll((long long)mq) - 1);
          mq &= mq - 1;
          met = ballot(boxes_meet(ep, one)) & mp;
        }
      }
    }
    if (met) touching |= 1ull << l;
  }
  if (live) out[k] = r | ((touching >> lane) & 1ull ? SCCG_REL_TOUCHES : 0u);
}

hipError_t launch_relate(const Polys& A, const Polys& B, const Meta* metaA, const Meta* metaB, const int64_t* areaA,
                         const int64_t* areaB, int64_t n_pairs, const int32_t* pa, const int32_t* pb,
                         const int64_t* inter, uint32_t* out, uint32_t* err, hipStream_t s) {
  if (n_pairs <= 0) return hipSuccess;
  int per = kWave;
  while (per > 1 && n_pairs < (int64_t)per * 8192) per >>= 1;  // 8192 waves fill the chip
  for_slices(n_pairs, 256 / kWave * per, [&](int64_t first, unsigned blocks) {
    hipLaunchKernelGGL(k_relate, dim3(blocks), dim3(256), 0, s, A, B, metaA, metaB, areaA, areaB, n_pairs, pa, pb, inter,
                       out, err, per, first);
  });
  return hipGetLastError();
}

}  // namespace sccg
