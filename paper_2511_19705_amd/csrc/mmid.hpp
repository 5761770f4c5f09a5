// Middle factor of the gradient's way through rho(P) (paper Sec. 4.1: the squared norms of the inverse transform weigh the
// groups' squared maxima), from the partial headers of the loss pass.  One body, two users: launches of its own and of
// what follows the loss pass of a single matrix, and the gradient pass by records.
#pragma once
#include "loss_reduce.hpp"

namespace cafeq {

// workgroups whose chunk of macro-tiles intersects segment `seg`: [lo, hi)
// (the divisions, a few hundred instructions each in 64 bits, in 32 where they fit)
__device__ __forceinline__ void seg_wg_range(int64_t seg, int64_t mt_per_seg, int64_t n_mt, int nwg, int* lo, int* hi) {
  if (uint64_t(n_mt) * uint64_t(nwg + 1) < (uint64_t(1) << 32)) {
    const uint32_t n = uint32_t(n_mt), g = uint32_t(nwg), t0 = uint32_t(seg * mt_per_seg), t1 = t0 + uint32_t(mt_per_seg);
    // the last workgroup that begins at or before t0, the first that begins at or behind t1: w n / g rounded down is
    // below t where w n < t g
    const uint32_t a = ((t0 + 1) * g - 1) / n, b = (t1 * g + n - 1) / n;
    *lo = int(a < g ? a : g - 1);
    *hi = int(b < g ? b : g);
    return;
  }
  const int64_t t0 = seg * mt_per_seg, t1 = t0 + mt_per_seg;
  int a = int((t0 * nwg) / n_mt);
  while (a > 0 && chunk_begin(a, n_mt, nwg) > t0) --a;
  while (a + 1 < nwg && chunk_begin(a + 1, n_mt, nwg) <= t0) ++a;
  int b = a;
  while (b < nwg && chunk_begin(b, n_mt, nwg) < t1) ++b;
  *lo = a;
  *hi = b;
}

// v[axis index] = beta * sum over partials of the group's sum a^2, expanded per index, then
// Mmid_b = diag(v_b) P_b (scale_rows) or P_b diag(v_b).  For AXIS_ROW with rep > 1 the rep
// row-blocks of a transform block add up.   grid: nb transform blocks.
struct VArgs {
  const float* slot_hdr;
  int64_t mt_per_seg, n_mt;
  int nwg;
  int K, L, G, rep;
  float beta;
  const float* P;
  int scale_rows;
  float* Mmid;
};
constexpr int kMmidParts = 4;   // workgroups per block in the middle factor of the rho path
// (part of nparts: the workgroup scales that share of the block's elements; every part forms the same sums)
__device__ __forceinline__ void build_mmid_body(const VArgs& a, const int b, const int part, const int nparts) {
  __shared__ float v[256];
  __shared__ int rng[2];
  const int K = a.K, n = threadIdx.x;   // K <= 256 <= blockDim.x: thread n owns index n
  double acc = 0;
  for (int q = b * a.rep; q < (b + 1) * a.rep; ++q) {
    // the K axis indices of a row-block lie in one segment (L is a multiple of K): its range of
    // workgroups is found once (64-bit divisions) and shared
    const int64_t seg = (int64_t(q) * K) / a.L;
    if (n == 0) {
      int lo, hi;
      seg_wg_range(seg, a.mt_per_seg, a.n_mt, a.nwg, &lo, &hi);
      rng[0] = lo; rng[1] = hi;
    }
    __syncthreads();
    const int lo = rng[0], hi = rng[1];
    if (n < K) {
      const int gi = int(((int64_t(q) * K + n) % a.L) / a.G);
      const float* h0 = a.slot_hdr + seg * kHdrFloats + kHdrVa2 + gi;
      // eight requests in flight; the additions keep the order of the workgroups
      int w = lo;
      for (; w + 8 <= hi; w += 8) {
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = h0[int64_t(w + u) * kHdrFloats];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += t[u];
      }
      for (; w < hi; ++w) acc += h0[int64_t(w) * kHdrFloats];
    }
    __syncthreads();
  }
  if (n < K) v[n] = float(acc * a.beta);
  __syncthreads();
  const float* Pb = a.P + size_t(b) * K * K;
  float* Mb = a.Mmid + size_t(b) * K * K;
  // K * K / nparts elements, four per thread and step (K is a multiple of 32: rows are multiples of 4)
  const int per = K * K / nparts, e0 = part * per;
  for (int i = e0 + 4 * int(threadIdx.x); i < e0 + per; i += 4 * int(blockDim.x)) {
    const float4 pv = *reinterpret_cast<const float4*>(Pb + i);
    float4 o;
    if (a.scale_rows) {
      const float f = v[i / K];
      o = make_float4(pv.x * f, pv.y * f, pv.z * f, pv.w * f);
    } else {
      const int c = i % K;
      o = make_float4(pv.x * v[c], pv.y * v[c + 1], pv.z * v[c + 2], pv.w * v[c + 3]);
    }
    *reinterpret_cast<float4*>(Mb + i) = o;
  }
}

// L: axis indices per segment of the loss pass
inline VArgs mmid_args(const CoreParams& ploss, int K, int L, int G, const float* P, int scale_rows, float* Mmid) {
  VArgs a;
  a.slot_hdr = ploss.slot_hdr; a.mt_per_seg = ploss.mt_per_seg; a.n_mt = ploss.n_mt; a.nwg = ploss.nwg;
  a.K = K; a.L = L; a.G = G; a.rep = ploss.rep; a.beta = ploss.beta; a.P = P;
  a.scale_rows = scale_rows; a.Mmid = Mmid;
  return a;
}

}  // namespace cafeq
