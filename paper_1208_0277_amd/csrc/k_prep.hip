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
constexpr int kRow = 16;        // lanes per ring (a DPP row)
constexpr int kRowChunks = 4;   // loads of a lane in flight
constexpr int kRowStep = kRow * kRowChunks;

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
__device__ __forceinline__ uint64_t row_sum64(uint64_t v) {
  for (int d = 1; d < kRow; d <<= 1) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, d, kWave);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), d, kWave);
    v += ((uint64_t)hi << 32) | lo;
  }
  return v;
}

// Extents, and kArea |shoelace|/2 (Section 3.2's area formula), of the rings
// of one or two sets.  Twice the signed area is summed as (x + x') (y' - y)
// over the edges, x relative to the first vertex, modulo 2^32: exact for a
// ring at most kMaxSide wide and tall; a larger one has it summed again
// modulo 2^64, in which twice the area (at most 2^63 in size) is exact.
template <bool kArea>
__global__ void __launch_bounds__(256) k_meta_rows(Polys A, Meta* metaA, int64_t* areaA, Polys B, Meta* metaB,
                                                   int64_t* areaB, uint32_t* err) {
  int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kRow;
  const int j = (int)(threadIdx.x % kRow);
  const bool second = k >= A.n;
  if (second) k -= A.n;
  if (second && k >= B.n) return;
  const int64_t* off = second ? B.off : A.off;
  const int64_t o = off[k], nv = off[k + 1] - o;
  const int2* R = (second ? B.xy : A.xy) + o;
  int32_t x0 = INT_MAX, y0 = INT_MAX, nx1 = INT_MAX, ny1 = INT_MAX;
  uint32_t tn = 0;
  int2 f = make_int2(0, 0);
  if (kArea && nv > 0) f = R[0];
  for (int64_t base = 0; base < nv; base += kRowStep) {
    const RowChunk r = row_load<kArea>(R, nv, base, j);
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
  const Meta m{row_min(x0), row_min(y0), ~row_min(nx1), ~row_min(ny1)};
  const bool empty = nv <= 0;
  const bool bad = !empty && (m.x0 < -kMaxCoord || m.y0 < -kMaxCoord || m.x1 > kMaxCoord || m.y1 > kMaxCoord);
  int64_t area = 0;
  if (kArea && !empty && !bad) {
    if (side_u(m.x0, m.x1) <= (uint32_t)kMaxSide && side_u(m.y0, m.y1) <= (uint32_t)kMaxSide) {
      const int32_t t = (int32_t)row_sum(tn);
      area = (t < 0 ? -(int64_t)t : (int64_t)t) / 2;
    } else {
      uint64_t tw = 0;
      for (int64_t base = 0; base < nv; base += kRowStep) {
        const RowChunk r = row_load<true>(R, nv, base, j);
        for (int c = 0; c < kRowChunks; ++c)
          tw += (uint64_t)((int64_t)r.v[c].x * r.s[c].y) - (uint64_t)((int64_t)r.s[c].x * r.v[c].y);
      }
      const uint64_t t = row_sum64(tw);
      area = (int64_t)(((int64_t)t < 0 ? 0 - t : t) / 2);
    }
  }
  if (j != 0) return;
  if (bad) latch_error(err, kErrCoord);
  const bool none = empty || bad;
  *reinterpret_cast<int4*>((second ? metaB : metaA) + k) =
      none ? make_int4(INT_MAX, INT_MAX, INT_MIN, INT_MIN) : make_int4(m.x0, m.y0, m.x1, m.y1);
  if (kArea) (second ? areaB : areaA)[k] = area;
}

hipError_t launch_poly_meta(const Polys& A, Meta* metaA, int64_t* areaA, const Polys& B, Meta* metaB, int64_t* areaB,
                            uint32_t* err, hipStream_t s) {
  if (A.n + B.n <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)(((A.n + B.n) * kRow + 255) / 256);
  if (areaA)
    hipLaunchKernelGGL(k_meta_rows<true>, dim3(blocks), dim3(256), 0, s, A, metaA, areaA, B, metaB, areaB, err);
  else
    hipLaunchKernelGGL(k_meta_rows<false>, dim3(blocks), dim3(256), 0, s, A, metaA, areaA, B, metaB, areaB, err);
  return hipGetLastError();
}

// ---------------------------------------------------------------- validation
// -1 as the largest unsigned value: what the smallest bad index is taken from,
// and what is left when there is none
__global__ void k_validate_init(unsigned long long* first_bad) { *first_bad = ~0ull; }

__global__ void __launch_bounds__(256) k_validate(Polys P, unsigned long long* first_bad) {
  const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kRow;
  const int j = (int)(threadIdx.x % kRow);
  bool bad = false;
  if (k < P.n) {
    const int64_t o = P.off[k], nv = P.off[k + 1] - o;
    bad = nv < 4;
    for (int64_t base = 0; base < nv; base += kRowStep) {
      const RowChunk r = row_load<true>(P.xy + o, nv, base, j);
#pragma unroll
      for (int c = 0; c < kRowChunks; ++c) bad |= (r.v[c].x != r.s[c].x) & (r.v[c].y != r.s[c].y);
    }
  }
  // the wave's rings stand in order: its first bad lane has its smallest index
  const uint64_t m = ballot(bad);
  if (m && lane_id() == __ffsll((long long)m) - 1 &&
      (unsigned long long)k < __hip_atomic_load(first_bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMin(first_bad, (unsigned long long)k);
}

hipError_t launch_validate(const Polys& P, int64_t* first_bad, hipStream_t s) {
  auto* fb = reinterpret_cast<unsigned long long*>(first_bad);
  hipLaunchKernelGGL(k_validate_init, dim3(1), dim3(1), 0, s, fb);
  if (P.n > 0)
    hipLaunchKernelGGL(k_validate, dim3((unsigned)((P.n * kRow + 255) / 256)), dim3(256), 0, s, P, fb);
  return hipGetLastError();
}

// ------------------------------------------------------------------- Jaccard
// Per-set sums of Eq. 1 over the pairs of each set; J' by the exact ratio
// sum of fix192.h.  Workgroups claim chunks of kJacChunk consecutive pairs
// of the whole pair range, so that a large set is shared by many
// workgroups and many small sets by one.  For each set a chunk overlaps,
// the workgroup reduces its part and adds it to the set's accumulator:
// 64-bit atomics for the integer sums, and for the Fix192 ratio sum six
// 32-bit limbs, each added into a 64-bit counter (carry-save: a set gets at
// most 2^31 / kJacChunk + 1 additions, far from overflowing a counter).
// Integer and fixed-point addition do not depend on order, so the result is
// the same bits as any sequential sum.  A second pass normalizes the limbs
// and divides.
constexpr int kJacChunk = 4096;

__global__ void k_jaccard_clear(JacAcc* acc, int64_t n_sets, unsigned long long* next) {
  unsigned long long* w = reinterpret_cast<unsigned long long*>(acc);
  const int64_t n = n_sets * (int64_t)(sizeof(JacAcc) / 8);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    w[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *next = 0;
}

__global__ void __launch_bounds__(256) k_jaccard_chunks(int64_t n_sets, const int64_t* set_off,
                                                        const int64_t* inter, const int64_t* uni, uint32_t flags,
                                                        bool want_jp, JacAcc* acc, unsigned long long* next) {
  __shared__ uint64_t red[6][256];
  __shared__ int64_t chunk_s;
  const bool include_zero = (flags & SCCG_J_INCLUDE_ZERO) != 0;
  const int64_t base = set_off[0], end = set_off[n_sets];  // the pairs of all sets
  const int64_t n_chunks = (end - base + kJacChunk - 1) / kJacChunk;
  const int tid = threadIdx.x;
  for (;;) {
    if (tid == 0) chunk_s = (int64_t)atomicAdd(next, 1ull);
    __syncthreads();
    const int64_t chunk = chunk_s;
    __syncthreads();
    if (chunk >= n_chunks) break;
    const int64_t c0 = base + chunk * kJacChunk, c1 = min(c0 + (int64_t)kJacChunk, end);
    // the set holding pair c0: the last s with set_off[s] <= c0
    int64_t lo = 0, hi = n_sets - 1;
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) / 2;
      if (set_off[mid] <= c0) lo = mid;
      else hi = mid - 1;
    }
    for (int64_t s = lo; s < n_sets; ++s) {
      const int64_t o0 = max(set_off[s], c0), o1 = min(set_off[s + 1], c1);
      uint64_t si = 0, su = 0, nn = 0;
      Fix192 fx;
      for (int64_t k = o0 + tid; k < o1; k += blockDim.x) {
        const int64_t I = inter[k], U = uni[k];
        if (!include_zero && I == 0) continue;
        si += (uint64_t)I;
        su += (uint64_t)U;
        nn += 1;
        if (want_jp && U > 0) fx.add_ratio((double)I / (double)U);
      }
      red[0][tid] = si;
      red[1][tid] = su;
      red[2][tid] = nn;
      red[3][tid] = fx.w[0];
      red[4][tid] = fx.w[1];
      red[5][tid] = fx.w[2];
      __syncthreads();
      for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if (tid < h) {
          red[0][tid] += red[0][tid + h];
          red[1][tid] += red[1][tid + h];
          red[2][tid] += red[2][tid + h];
          Fix192 x, y;
          x.w[0] = red[3][tid]; x.w[1] = red[4][tid]; x.w[2] = red[5][tid];
          y.w[0] = red[3][tid + h]; y.w[1] = red[4][tid + h]; y.w[2] = red[5][tid + h];
          x.add(y);
          red[3][tid] = x.w[0]; red[4][tid] = x.w[1]; red[5][tid] = x.w[2];
        }
        __syncthreads();
      }
      if (tid == 0 && red[2][0] != 0) {
        JacAcc& A = acc[s];
        atomicAdd(&A.si, (unsigned long long)red[0][0]);
        atomicAdd(&A.su, (unsigned long long)red[1][0]);
        atomicAdd(&A.nn, (unsigned long long)red[2][0]);
        for (int k = 0; k < 3; ++k) {
          const uint64_t w = red[3 + k][0];
          if (w & 0xffffffffull) atomicAdd(&A.limb[2 * k], (unsigned long long)(w & 0xffffffffull));
          if (w >> 32) atomicAdd(&A.limb[2 * k + 1], (unsigned long long)(w >> 32));
        }
      }
      __syncthreads();
      if (set_off[s + 1] >= c1) break;
    }
  }
}

__global__ void k_jaccard_final(int64_t n_sets, const JacAcc* acc, bool want_jp, int64_t* sum_i, int64_t* sum_u,
                                int64_t* n_contrib, double* jout, double* jprime) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_sets) return;
  const JacAcc A = acc[s];
  const int64_t tI = (int64_t)A.si, tU = (int64_t)A.su, tn = (int64_t)A.nn;
  sum_i[s] = tI;
  sum_u[s] = tU;
  n_contrib[s] = tn;
  jout[s] = tU > 0 ? (double)tI / (double)tU : 0.0;
  if (want_jp) {
    // limb k weighs 2^(32 k): add them up with carries into three words
    Fix192 f;
    for (int k = 0; k < 6; ++k) {
      Fix192 t;
      const uint64_t v = A.limb[k];
      const int sh = 32 * k, w = sh >> 6, off = sh & 63;
      t.w[w] = v << off;
      if (off && w + 1 < 3) t.w[w + 1] = v >> (64 - off);
      f.add(t);
    }
    jprime[s] = tn > 0 ? f.to_double() / (double)tn : 0.0;
  }
}

hipError_t launch_jaccard(int64_t n_sets, const int64_t* set_off, const int64_t* inter, const int64_t* uni,
                          uint32_t flags, int64_t* sum_i, int64_t* sum_u, int64_t* n_contrib, double* j,
                          double* jprime, JacAcc* acc, unsigned long long* next, int grid, hipStream_t s) {
  if (n_sets <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_jaccard_clear, dim3(256), dim3(256), 0, s, acc, n_sets, next);
  hipLaunchKernelGGL(k_jaccard_chunks, dim3(grid), dim3(256), 0, s, n_sets, set_off, inter, uni, flags,
                     jprime != nullptr, acc, next);
  hipLaunchKernelGGL(k_jaccard_final, dim3((unsigned)((n_sets + 255) / 256)), dim3(256), 0, s, n_sets, acc,
                     jprime != nullptr, sum_i, sum_u, n_contrib, j, jprime);
  return hipGetLastError();
}

}  // namespace sccg
