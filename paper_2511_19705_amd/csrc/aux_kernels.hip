// Small kernels around the fused core: squared norms of the inverse transform (the
// (M^-1)_{ij}^2 factors of the paper's surrogate, Sec. 4.1), fixed-order reduction of the
// per-workgroup partials and the k x k products of the gradient's path through M^-1.  All are off the bandwidth path (k x k sized per block).
#include <atomic>
#include "cafeq_internal.hpp"
#include "xform_core.hpp"
#include "loss_reduce.hpp"
#include "mmid.hpp"
#include "ns_inverse.hpp"

namespace cafeq {

namespace {

// What the loss pass needs of the transform besides the weights, in one launch: operand planes (SplitJob) and the
// squared norms of the inverse (RhoJob).  Workgroups of 1024 threads, one per (block, job); both kinds read a block's
// k x k floats once, with every request in flight before the first use, so a workgroup costs one memory latency and not
// one per 32 x k stage.  Measured against a split launch that walked the stages (and scanned the block once more for its
// magnitude) after a rho launch of 256 threads per block: 144 blocks of 64
// 6.9 + 5.7 -> 6.5 us, 72 blocks of 128 10.9 + 8.1 -> 8.2 us, 8 blocks of 32 3.8 + 2.9 -> 3.6 us.
constexpr int kSplitThreads = 1024;

// Operand planes of the fused core.  Element [out][in] of the k x k operand -- src_b (trans == 0) or
// src_b^T (trans == 1) -- is split exactly into bfloat16 parts x = hi + mid + lo (+ a residual below
// 2^-24 |x|) and stored in the order the core streams it through its LDS ring:
//   dst[b][stage = in / 32][part][out][32 inputs of the stage]
// with the 32 inputs of a row arranged as four 16-byte chunks (MFMA step c2 = (in % 32) / 16, lane
// half h -> chunk 2*c2 + h, holding inputs 16*c2 + 8u + 4h + e at position 4u + e), the chunk stored
// at chunk ^ ((out >> 2) & 3) (LDS bank swizzle).
struct SplitJob { const float* src; uint16_t* dst; int trans, nplanes; float* fscale; int natural, texp, minus_one; };   // fscale, texp: see below
// A job with fscale != null writes two (or three: nplanes) float16 planes instead: the block is first scaled by the power of
// two that puts its largest magnitude into [2^texp, 2^(texp+1)) (14: the low parts stay normal numbers; 4: sums of
// 128 products with operands below 2^4 stay below 2^16 -- the matrix cores take denormal float16 inputs exactly), then
// x = hi + lo (+ a third) with the parts rounded to nearest; fscale[b] receives the factor that undoes the scale.
// minus_one (K = 256, bfloat16 planes): of src_b - I.
//
// rho[b*K + j]: squared norm of row j (by_row) or column j of P_b, summed in float64.
// With rG != null the workgroup also writes the sums of rho over groups of G axis indices (what rho_group_kernel
// computes, lanes interleaved over a group's indices, then a wave sum):
//   G <= K, G | K, nbk = 1: rG[(b rep + r) (K / G) + q] = sum over indices q G .. q G + G - 1 of block b, for each
//                           of the rep row-blocks that share the block;
//   G = nbk K <= 256, rep = 1: rG[workgroup] = sum over its nbk blocks (consecutive ones).
struct RhoJob { const float* P; float* rho; float* rG; int by_row, G, rep, nbk; };
struct SplitJobs {
  SplitJob job[4]; RhoJob rho[2]; int njobs, nrho, nb;
  float* hdr; int64_t nhdr;     // partial headers to reset (may be null)
};

template <int K>
__device__ __forceinline__ void rho_body(const RhoJob& jb, const int nb, double* part /* [16][K] */, float* line /* [256] */) {
  constexpr int LPR = K / 4, ROWS = kSplitThreads / LPR, NQ = K / ROWS > 0 ? K / ROWS : 1;   // lanes per row, rows per pass
  const int tid = threadIdx.x, c = 4 * (tid % LPR), r0 = tid / LPR, lane = tid % kWave, wave = tid / kWave;
  if (int64_t(blockIdx.x) * jb.nbk >= nb) return;
  for (int bb = 0; bb < jb.nbk; ++bb) {
    const size_t b = size_t(blockIdx.x) * jb.nbk + bb;
    const float* Pb = jb.P + b * K * K;
    float4 u[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int r = r0 + q * ROWS;
      u[q] = r < K ? *reinterpret_cast<const float4*>(Pb + r * K + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (jb.by_row) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        double t = double(u[q].x) * u[q].x + double(u[q].y) * u[q].y + double(u[q].z) * u[q].z + double(u[q].w) * u[q].w;
#pragma unroll
        for (int o = 1; o < LPR; o *= 2) t += __shfl_xor(t, o);
        const int r = r0 + q * ROWS;
        if (c == 0 && r < K) { jb.rho[b * K + r] = float(t); if (jb.rG) line[bb * K + r] = float(t); }   // (rG set: nbk K <= 256)
      }
    } else {
      double t[4] = {0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        t[0] += double(u[q].x) * u[q].x; t[1] += double(u[q].y) * u[q].y;
        t[2] += double(u[q].z) * u[q].z; t[3] += double(u[q].w) * u[q].w;
      }
#pragma unroll
      for (int o = LPR; o < kWave; o *= 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] += __shfl_xor(t[e], o);
      if (lane < LPR)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[wave * K + c + e] = t[e];
      __syncthreads();
      if (tid < K) {
        double s = part[tid];
#pragma unroll
        for (int w = 1; w < kSplitThreads / kWave; ++w) s += part[w * K + tid];
        jb.rho[b * K + tid] = float(s);
        if (jb.rG) line[bb * K + tid] = float(s);
      }
    }
    __syncthreads();
  }
  if (jb.rG == nullptr) return;                  // uniform
  if (jb.nbk > 1) {
    if (wave == 0) {
      float acc = 0.f;
      for (int e = lane; e < jb.G; e += kWave) acc += line[e];
      acc = wave_sum(acc);
      if (lane == 0) jb.rG[blockIdx.x] = acc;
    }
    return;
  }
  const int ng = K / jb.G;
  for (int q = wave; q < ng; q += kSplitThreads / kWave) {
    float acc = 0.f;
    for (int e = lane; e < jb.G; e += kWave) acc += line[q * jb.G + e];
    acc = wave_sum(acc);
    if (lane == 0)
      for (int r = 0; r < jb.rep; ++r) jb.rG[(size_t(blockIdx.x) * jb.rep + r) * ng + q] = acc;
  }
}

// grid: (nb, njobs + nrho, z): with z > 1 (few blocks, and blocks of 256, which a workgroup cannot hold in registers) the
// K / 32 stages of a block go to a workgroup each.
template <int K>
__global__ __launch_bounds__(kSplitThreads) void split_planes_kernel(const SplitJobs js) {
  // stages' planes are assembled in LDS in their final order and leave as whole 16-byte vectors
  constexpr int kLdsB = K == 32 ? 33 * 1024 : 64 * 1024;
  __shared__ __align__(16) unsigned char lds[kLdsB];
  __shared__ float wmx[kSplitThreads / 64], line[256];
  constexpr int NST = K / 32, QPS = K * 8;                                 // stages, quads a stage
  constexpr int NQ = K == 256 ? QPS / kSplitThreads : (K * K / 4 + kSplitThreads - 1) / kSplitThreads;   // quads a thread
  const int tid = threadIdx.x;
  // partial headers that no workgroup of the core writes (slots nobody owns) must read as empty
  if (js.hdr) {
    const int64_t nthr = int64_t(gridDim.x) * gridDim.y * gridDim.z * kSplitThreads;
    for (int64_t i = ((int64_t(blockIdx.z) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * kSplitThreads + tid;
         i < js.nhdr; i += nthr)
      js.hdr[i] = (i % kHdrFloats) == kHdrMref ? -INFINITY : 0.f;
  }
  if (int(blockIdx.y) >= js.njobs) {
    if (blockIdx.z == 0) rho_body<K>(js.rho[int(blockIdx.y) - js.njobs], js.nb, reinterpret_cast<double*>(lds), line);
    return;
  }
  const SplitJob jb = js.job[blockIdx.y];
  const int nplanes = jb.nplanes;
  const float* sb = jb.src + size_t(blockIdx.x) * K * K;
  const bool whole = K < 256 && gridDim.z == 1;
  const int stage0 = whole ? 0 : int(blockIdx.z), nquad = whole ? K * K / 4 : QPS;
  // a quad: four inputs that are adjacent in the plane (e = 0..3 of one (row, step, half, u)): one 128-bit load (or four
  // coalesced loads of a transposed source) and one 64-bit LDS store per plane
  float4 x[NQ];
  float m = 0.f;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = tid + q * kSplitThreads, stage = stage0 + i / QPS, qd = i % QPS;
    x[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < nquad) {
      if (jb.trans) {
        const float* p = sb + size_t(32 * stage + 4 * (qd / K)) * K + qd % K;
        x[q] = make_float4(p[0], p[K], p[2 * K], p[3 * K]);
      } else {
        x[q] = *reinterpret_cast<const float4*>(sb + size_t(qd >> 3) * K + 32 * stage + 4 * (qd & 7));
      }
    }
  }
  if constexpr (K == 256) {
    if (jb.minus_one) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int qd = tid + q * kSplitThreads, d = jb.trans ? qd % K - 32 * stage0 - 4 * (qd / K) : (qd >> 3) - 32 * stage0 - 4 * (qd & 7);
        x[q].x -= d == 0 ? 1.f : 0.f; x[q].y -= d == 1 ? 1.f : 0.f; x[q].z -= d == 2 ? 1.f : 0.f; x[q].w -= d == 3 ? 1.f : 0.f;
      }
    }
  }
  float hsc = 1.f;   // float16 job: the block's scale
  if (jb.fscale) {
    // (an infinite entry must not set the scale: the block's other outputs would be scaled away.  Looked for only where there is one)
    for (int finite = 0; finite < 2; ++finite) {
      m = 0.f;
      auto take = [&](float4 v) {
        if (finite) {
          for (float e : {v.x, v.y, v.z, v.w})
            if (fabsf(e) < INFINITY) m = fmaxf(m, fabsf(e));
        } else {
          m = fmaxf(fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w)));
        }
      };
      if (whole) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) take(x[q]);
      } else {
        for (int e = tid * 4; e < K * K; e += kSplitThreads * 4) take(*reinterpret_cast<const float4*>(sb + e));
      }
      m = cluster_allmax<64>(m);
      if (finite) __syncthreads();                                         // (the maxima before have been read)
      if ((tid & 63) == 0) wmx[tid >> 6] = m;
      __syncthreads();
      m = 0.f;
#pragma unroll
      for (int i = 0; i < kSplitThreads / 64; ++i) m = fmaxf(m, wmx[i]);
      if (m < INFINITY) break;                                             // (uniform)
    }
    int ex = int(__float_as_uint(m) >> 23);
    ex = ex < 32 ? 32 : (ex > 254 ? 254 : ex);
    hsc = __uint_as_float(uint32_t(254 + jb.texp - ex) << 23);             // 2^(texp - (ex - 127))
    if (tid == 0 && blockIdx.z == 0) jb.fscale[blockIdx.x] = __uint_as_float(uint32_t(ex - jb.texp) << 23);
  }
  const int spr = kLdsB / (nplanes * K * 64);                              // stages that fit the LDS (K = 256, three planes: one)
  const int nstw = whole ? NST : 1;
  for (int s0 = 0; s0 < nstw; s0 += spr) {
    if (s0 > 0) __syncthreads();                                           // the stages before have left
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int i = tid + q * kSplitThreads, sr = i / QPS - s0, qd = i % QPS;
      if (i >= nquad || sr < 0 || sr >= spr) continue;
      const int out = jb.trans ? qd % K : qd >> 3, wq = jb.trans ? qd / K : qd & 7;
      // quad wq holds inputs 4 wq .. 4 wq + 3 of the stage = 16 c2 + 8 u + 4 hh + e; with the natural order the
      // lane half takes eight consecutive inputs, i.e. the two middle bits swap their roles
      const int c2 = wq >> 2, u = jb.natural ? (wq & 1) : (wq >> 1) & 1, hh = jb.natural ? (wq >> 1) & 1 : (wq & 1);
      const int chunk = (2 * c2 + hh) ^ ((out >> 2) & 3);
      uint16_t* at = reinterpret_cast<uint16_t*>(lds) + sr * nplanes * K * 32 + out * 32 + chunk * 8 + 4 * u;
      float y[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
      if (jb.fscale) {
        uint32_t hi[4], lo[4], lo2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float z = y[e] * hsc;
          const _Float16 a = _Float16(z);
          const float r = z - float(a);
          const _Float16 b = _Float16(r);
          hi[e] = __builtin_bit_cast(uint16_t, a);
          lo[e] = __builtin_bit_cast(uint16_t, b);
          lo2[e] = __builtin_bit_cast(uint16_t, _Float16(r - float(b)));
        }
        *reinterpret_cast<uint2*>(at) = make_uint2(hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16));
        *reinterpret_cast<uint2*>(at + K * 32) = make_uint2(lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16));
        if (nplanes == 3) *reinterpret_cast<uint2*>(at + 2 * K * 32) = make_uint2(lo2[0] | (lo2[1] << 16), lo2[2] | (lo2[3] << 16));
        continue;
      }
      for (int pl = 0; pl < nplanes; ++pl) {
        uint32_t part[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t bits = __float_as_uint(y[e]);
          bits += 0x7FFFu + ((bits >> 16) & 1u);          // round to nearest even
          part[e] = bits >> 16;
          y[e] -= __uint_as_float(part[e] << 16);
        }
        *reinterpret_cast<uint2*>(at + pl * K * 32) = make_uint2(part[0] | (part[1] << 16), part[2] | (part[3] << 16));
      }
    }
    __syncthreads();
    const int ns = nstw - s0 < spr ? nstw - s0 : spr;
    const uint4* s4 = reinterpret_cast<const uint4*>(lds);
    uint4* d4 = reinterpret_cast<uint4*>(jb.dst + (size_t(blockIdx.x) * NST + stage0 + s0) * nplanes * K * 32);
    for (int e = tid; e < ns * nplanes * K * 4; e += kSplitThreads) d4[e] = s4[e];
  }
}

// rG[gi] = sum of rho over the axis indices of group gi (axis index a -> block (a/K)/rep, a%K), wpg waves per group (1
// or the whole workgroup).  Groups that launch_split_planes_multi's rho jobs do not cover: longer than 256, or across
// row-blocks that share a block.  A whole channel is one group: with one wave its sum was a chain of up to naxis / 64
// loads (61 us at 9216; now 4.9 us).
constexpr int kRhoGroupWaves = 16;
__global__ __launch_bounds__(kRhoGroupWaves * kWave) void rho_group_kernel(const float* __restrict__ rho, int lk, int rep,
                                                                          int G, int64_t ngroups, int wpg,
                                                                          float* __restrict__ rG) {
  __shared__ double part[kRhoGroupWaves];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, per = kRhoGroupWaves / wpg;
  const int64_t gi = int64_t(blockIdx.x) * per + (wpg == 1 ? wave : 0);
  const int nthr = wpg * kWave, t0 = wpg == 1 ? lane : int(threadIdx.x);
  double acc = 0;
  if (gi < ngroups) {
#pragma unroll 8
    for (int e = t0; e < G; e += nthr) {
      const int64_t a = gi * G + e;
      const unsigned q = unsigned(a >> lk), b = rep == 1 ? q : q / unsigned(rep);
      acc += rho[(int64_t(b) << lk) + (a & ((1 << lk) - 1))];
    }
  }
#pragma unroll
  for (int o = 1; o < kWave; o *= 2) acc += __shfl_xor(acc, o);
  if (wpg > 1) {
    if (lane == 0) part[wave] = acc;
    __syncthreads();
    acc = part[0];
#pragma unroll
    for (int w = 1; w < kRhoGroupWaves; ++w) acc += part[w];
    if (threadIdx.x == 0) rG[gi] = float(acc);
  } else if (lane == 0 && gi < ngroups) {
    rG[gi] = float(acc);
  }
}

// ---------------------------------------------------------------------------------------
// reduction of the per-(workgroup, segment) partials
// ---------------------------------------------------------------------------------------
struct ReduceArgs {
  const float* slot_grad;
  const float* slot_hdr;
  int64_t mt_per_seg, n_mt;   // of the pass that wrote the partials
  int nwg, nseg;
  int K, rep;
  int seg_len;           // axis indices per segment of that pass
  int part_floats;       // floats of one partial
  int msplit;            // 1: a partial holds whole blocks, [seg_len outputs][K inputs];
                         // 2: K == 256 in halves of the inputs, [256 outputs][128 inputs], segment 2 q + half
  int transpose_out;     // 1: out[m][j] = acc[j][m]
  float t;               // kLossLse: temperature; scale of a partial = exp(t (m_ref - m*)) / S
  const double* lse_ms;  // kLossLse: [0] = m*, [1] = S  (null for kLossSur)
  const float* member_ref;  // kLossLse, two-pass gradient: every partial is relative to this value
  float* out;            // [nb][K][K]
};

// grid: (nb transform blocks, K*K/1024).  out_b = sum over the rep row-blocks q of block b, and
// over the partials of q's segment, in fixed order; each thread owns four consecutive inputs of one
// output row, each workgroup 1024 elements that lie in one partial layout (one half when msplit == 2).
struct ReduceJobs { ReduceArgs job[2]; };   // grid.z picks the job (the two members of a pair in one launch)
__device__ __forceinline__ void reduce_grad_body(const ReduceArgs& a, const int b, const int by) {
  constexpr int kBatch = 64;
  __shared__ const float* src[kBatch];
  __shared__ float scl[kBatch];
  __shared__ int rng_lo, rng_hi;
  const int K = a.K;
  // this workgroup's 1024 elements: rows of KMr inputs inside one half
  const int KMr = a.msplit == 2 ? 128 : K;
  const int rows_per_wg = 1024 / KMr;                       // K = 32: one workgroup covers the block
  const int nyh = K / rows_per_wg > 0 ? K / rows_per_wg : 1;
  const int half = by / nyh, rg = by % nyh;
  const int j = rg * rows_per_wg + (threadIdx.x * 4) / KMr, ml = (threadIdx.x * 4) % KMr;
  const bool active = j < K;
  const int poff = j * KMr + ml;                            // offset inside a partial (plus the block's base)
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  // every partial of a two-pass member carries the same scale
  float sc_all = 1.f;
  if (a.lse_ms && a.member_ref) sc_all = float(exp(double(a.t) * (double(*a.member_ref) - a.lse_ms[0])) / a.lse_ms[1]);
  for (int q = b * a.rep; q < (b + 1) * a.rep; ++q) {
    int seg, base;
    if (a.msplit == 2) { seg = 2 * q + half; base = 0; }
    else { seg = int((int64_t(q) * K) / a.seg_len); base = int((int64_t(q) * K) % a.seg_len) * K; }
    if (threadIdx.x == 0) {
      int lo, hi;
      seg_wg_range(seg, a.mt_per_seg, a.n_mt, a.nwg, &lo, &hi);
      rng_lo = lo; rng_hi = hi;
    }
    __syncthreads();
    const int lo = rng_lo, hi = rng_hi;
    for (int w0 = lo; w0 < hi; w0 += kBatch) {
      const int n = hi - w0 < kBatch ? hi - w0 : kBatch;
      // the list of (partial, scale) pairs of this batch, one thread per entry
      if (int(threadIdx.x) < n) {
        const int64_t slot = int64_t(w0 + int(threadIdx.x)) + seg;
        float sc = sc_all;
        if (a.lse_ms && !a.member_ref)
          sc = float(exp(double(a.t) * (double(a.slot_hdr[slot * kHdrFloats + kHdrMref]) - a.lse_ms[0])) / a.lse_ms[1]);
        src[threadIdx.x] = a.slot_grad + slot * int64_t(a.part_floats) + base;
        scl[threadIdx.x] = sc;
      }
      __syncthreads();
      if (active) {
        // four partials in flight per thread; the additions keep the order of the list
        int s = 0;
        for (; s + 4 <= n; s += 4) {
          float4 v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4*>(src[s + u] + poff);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float sc = scl[s + u];
            acc.x += sc * v[u].x; acc.y += sc * v[u].y; acc.z += sc * v[u].z; acc.w += sc * v[u].w;
          }
        }
        for (; s < n; ++s) {
          const float4 v = *reinterpret_cast<const float4*>(src[s] + poff);
          const float sc = scl[s];
          acc.x += sc * v.x; acc.y += sc * v.y; acc.z += sc * v.z; acc.w += sc * v.w;
        }
      }
      __syncthreads();
    }
  }
  if (active) {
    float* dst = a.out + size_t(b) * K * K;
    const int m = half * 128 + ml;
    if (a.transpose_out) {
      dst[(m + 0) * K + j] = acc.x; dst[(m + 1) * K + j] = acc.y;
      dst[(m + 2) * K + j] = acc.z; dst[(m + 3) * K + j] = acc.w;
    } else {
      *reinterpret_cast<float4*>(dst + j * K + m) = acc;
    }
  }
}
__global__ __launch_bounds__(256) void reduce_grad_kernel(const ReduceJobs js) {
  reduce_grad_body(js.job[blockIdx.z], int(blockIdx.x), int(blockIdx.y));
}

__global__ __launch_bounds__(256) void build_mmid_kernel(const VArgs a) {
  build_mmid_body(a, int(blockIdx.x) / kMmidParts, int(blockIdx.x) % kMmidParts, kMmidParts);
}

// losses: fixed-order float64 sums over every partial header (loss_reduce.hpp), as a launch of its own
__global__ __launch_bounds__(kLossThreads) void reduce_losses_kernel(const LossArgs a) {
  __shared__ double red[5 * (kLossThreads / 64)];
  double m, s;
  reduce_losses_body<kLossThreads>(a, red, true, &m, &s);
}

// What follows the loss / gradient kernel of a single matrix whose gradient comes as partials, in one launch:
// the gradient reduction (nred_x x nred_y workgroups), the middle factor of the gradient's way through rho(P)
// (kMmidParts workgroups per block) and the loss reduction (one workgroup) read the same partials and do not depend
// on each other.
__global__ __launch_bounds__(256) void single_tail_kernel(const ReduceArgs ra, const VArgs va, const LossArgs la,
                                                          const int nred_x, const int nred_y, const int nb) {
  const int id = int(blockIdx.x), nred = nred_x * nred_y;
  if (id < nred) {
    reduce_grad_body(ra, id % nred_x, id / nred_x);
  } else if (id < nred + nb * kMmidParts) {
    build_mmid_body(va, (id - nred) / kMmidParts, (id - nred) % kMmidParts, kMmidParts);
  } else {
    __shared__ double red[5 * (kLossThreads / 64)];
    double m, sm;
    reduce_losses_body<kLossThreads>(la, red, true, &m, &sm);
  }
}

// ---------------------------------------------------------------------------------------
// batched k x k product  C_b = alpha * op(A_b) op(B_b) + beta * C_b   (64 x 64 tile / workgroup)
// ---------------------------------------------------------------------------------------
// What the update needs of the element's old state, requested before the products it follows (behind them every load
// waited for the stores of the element before it, which may alias: 16 latencies in a row, 32 us instead of 17 for the 72
// blocks of 128 of the 2B-shaped pair).
struct UpdateOld { float t, m, v; };
__device__ __forceinline__ UpdateOld update_load(const UpdateHook& u, size_t at) {
  UpdateOld o{0.f, 0.f, 0.f};
  if (u.T) {
    o.t = u.T[at];
    if (u.m) { o.m = u.m[at]; o.v = u.v[at]; }
  }
  return o;
}
// (the arithmetic of adam_kernel / div_dev_kernel and sgd_kernel, on the gradient still in its register)
__device__ __forceinline__ void update_store(const UpdateHook& u, size_t at, float g, const UpdateOld& o, float denom) {
  if (u.m) {
    const float mi = u.beta1 * o.m + u.omb1 * g;
    const float vi = u.beta2 * o.v + u.omb2 * g * g;
    u.m[at] = mi;
    u.v[at] = vi;
    u.T[at] = o.t - u.lr * (mi * u.c1) / (sqrtf(vi * u.c2) + u.eps);
  } else {
    const float gd = u.denom ? g / denom : g;
    u.T[at] = o.t - u.lr * gd;
  }
}

// On the matrix cores (v_mfma_f32_32x32x2_f32) for K a multiple of 64: one 64 x 64
// output tile per workgroup, four waves of one 32 x 32 tile each, the operand panels staged in
// LDS as [contraction index][64 tile indices] (row stride 65 floats: transposing stores, whose
// lanes walk the contraction index, and the MFMA operand reads, whose lane halves take rows l
// and l+1, both stay clear of bank conflicts).  Contraction in chunks of CH = min(K, 128): the blocks of
// 128 the learning loops run on take one chunk -- every load of the workgroup is in flight at once and
// there is one barrier -- at 65 KB of LDS, two workgroups per compute unit.
// KS = 2 (K = 256): the two chunks side by side, four waves each, and their sums added through LDS: where there are no more workgroups
// than compute units, the second chunk's loads and products need not wait for the first's.  P^T G of 8 blocks 12.1 -> 10.7 us; the
// product by P^T behind it, which waits for the update's state as well, keeps 13.8 either way.
template <bool TA, bool TB, int CH, int KS = 1>
__global__ __launch_bounds__(256 * KS) void bgemm_mfma_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                          float* __restrict__ C, int K, float alpha, float beta,
                                                          const UpdateHook up) {
  constexpr int LD = 65;
  extern __shared__ __align__(16) float bsm[];
  const int part = KS == 2 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;   // its share of the contraction
  float* sa = bsm + part * (2 * CH * LD);
  float* sb = sa + CH * LD;
  const int tpr = K / 64;
  int b, tile;
  block_and_part(blockIdx.x, tpr * tpr, gridDim.x, &b, &tile);
  const int i0 = (tile / tpr) * 64, j0 = (tile % tpr) * 64;
  const float* Ab = A + size_t(b) * K * K;
  const float* Bb = B + size_t(b) * K * K;
  float* Cb = C + size_t(b) * K * K;
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6, ln = lane & 31, h = lane >> 5;
  const int wi = wave >> 1, wj = wave & 1;
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  // the old value of the output, where it is added to: requested before everything else
  float cold[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) cold[v] = 0.f;
  if (beta != 0.f && part == 0) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      cold[v] = Cb[(i0 + wi * 32 + 8 * (v / 4) + 4 * h + (v % 4)) * K + j0 + wj * 32 + ln];
  }
  UpdateOld old[16];
  if (up.T && part == 0) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      old[v] = update_load(up, size_t(b) * K * K + size_t(i0 + wi * 32 + 8 * (v / 4) + 4 * h + (v % 4)) * K + j0 + wj * 32 + ln);
  }
  const float denom = up.T && up.denom ? *up.denom : 1.f;
  for (int l0 = part * CH; l0 < K; l0 += KS * CH) {
    // sa[l][i] = op(A)[i0 + i][l0 + l];  sb[l][j] = op(B)[l0 + l][j0 + j]: four consecutive elements of the
    // operand's rows per load, all loads of the chunk issued before the first LDS store
    constexpr int NV = CH * 64 / 4 / 256;   // float4 per thread and panel
    float4 va[NV], vb[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int e = (tid + u * 256) * 4;
      if (TA) { const int l = e >> 6, i = e & 63; va[u] = *reinterpret_cast<const float4*>(Ab + (l0 + l) * K + i0 + i); }
      else    { const int i = e / CH, l = e % CH; va[u] = *reinterpret_cast<const float4*>(Ab + (i0 + i) * K + l0 + l); }
      if (TB) { const int j = e / CH, l = e % CH; vb[u] = *reinterpret_cast<const float4*>(Bb + (j0 + j) * K + l0 + l); }
      else    { const int l = e >> 6, j = e & 63; vb[u] = *reinterpret_cast<const float4*>(Bb + (l0 + l) * K + j0 + j); }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int e = (tid + u * 256) * 4;
      if (TA) { const int l = e >> 6, i = e & 63; float* d = sa + l * LD + i; d[0] = va[u].x; d[1] = va[u].y; d[2] = va[u].z; d[3] = va[u].w; }
      else    { const int i = e / CH, l = e % CH; float* d = sa + l * LD + i; d[0] = va[u].x; d[LD] = va[u].y; d[2 * LD] = va[u].z; d[3 * LD] = va[u].w; }
      if (TB) { const int j = e / CH, l = e % CH; float* d = sb + l * LD + j; d[0] = vb[u].x; d[LD] = vb[u].y; d[2 * LD] = vb[u].z; d[3 * LD] = vb[u].w; }
      else    { const int l = e >> 6, j = e & 63; float* d = sb + l * LD + j; d[0] = vb[u].x; d[1] = vb[u].y; d[2] = vb[u].z; d[3] = vb[u].w; }
    }
    __syncthreads();
    const float* pa = sa + h * LD + wi * 32 + ln;
    const float* pb = sb + h * LD + wj * 32 + ln;
    for (int s0 = 0; s0 < CH / 2; s0 += 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[2 * (s0 + u) * LD], pb[2 * (s0 + u) * LD], acc, 0, 0, 0);
    }
    if (KS == 1 && l0 + CH < K) __syncthreads();
  }
  if constexpr (KS == 2) {
    __syncthreads();
    float* sum = bsm + wave * 1024 + lane * 16;
    if (part == 1) {
#pragma unroll
      for (int q = 0; q < 4; ++q) *reinterpret_cast<float4*>(sum + 4 * (q ^ (lane & 3))) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    }
    __syncthreads();
    if (part == 1) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 t = *reinterpret_cast<const float4*>(sum + 4 * (q ^ (lane & 3)));
      acc[4 * q] += t.x; acc[4 * q + 1] += t.y; acc[4 * q + 2] += t.z; acc[4 * q + 3] += t.w;
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = i0 + wi * 32 + 8 * (v / 4) + 4 * h + (v % 4), j = j0 + wj * 32 + ln;
    const float g = alpha * acc[v] + (beta != 0.f ? beta * cold[v] : 0.f);
    if (up.T) {
      update_store(up, size_t(b) * K * K + size_t(i) * K + j, g, old[v], denom);
    } else {
      Cb[i * K + j] = g;
    }
  }
}

// The gradient's way through the inverse in one launch for blocks of 64: C = beta C + alpha (P^T G) P^T per block
// (Sec. 4.1 / 4.2: d/dT of a function of P = T^-1 is -P^T (d/dP) P^T), a workgroup of four waves of one 32 x 32 tile each, both
// products on v_mfma_f32_32x32x2_f32 in the arithmetic (and summation order) of bgemm_mfma_kernel.  P is staged once in LDS, row-major with a row stride of 65 floats, which serves the first product's A operand (lanes along a row) and
// the second's B operand (lanes along a column) without bank conflicts; G goes from memory straight into the
// registers of the wave that multiplies by it; X passes through LDS transposed.
// Bound: latency of load, LDS and the chain of matrix instructions.
constexpr int kChainLdX = 33;
constexpr size_t kChain64Lds = size_t(64 * 65 + 2 * 64 * kChainLdX) * sizeof(float);
__global__ __launch_bounds__(256) void bgemm_chain64_kernel(const float* __restrict__ P, const float* __restrict__ G, float* __restrict__ C,
                                                            float alpha, float beta, const UpdateHook up) {
  constexpr int K = 64, kChainLdP = K + 1, NT = 256;
  extern __shared__ __align__(16) float csm[];
  float* sp = csm;                          // P[r][c]
  float* sx = csm + K * kChainLdP;          // [2 row halves][l][32 rows]: X^T
  const int b = int(blockIdx.x);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 31, h = lane >> 5;
  const int wi = wave >> 1, wj = wave & 1;
  const float* Pb = P + size_t(b) * K * K;
  const float* Gb = G + size_t(b) * K * K;
  float* Cb = C + size_t(b) * K * K;
  // every load of the workgroup is requested before the first wait: P (for LDS), this wave's columns of G, and the
  // old value of the output where it is added to
  constexpr int NVP = K * K / 4 / NT;       // float4 of P per thread
  float4 vp[NVP];
#pragma unroll
  for (int u = 0; u < NVP; ++u) vp[u] = *reinterpret_cast<const float4*>(Pb + (tid + u * NT) * 4);
  float g[K / 2];
#pragma unroll
  for (int t = 0; t < K / 2; ++t) g[t] = Gb[(2 * t + h) * K + wj * 32 + ln];
  float cold[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) cold[v] = 0.f;
  if (beta != 0.f) {
#pragma unroll
    for (int v = 0; v < 16; ++v) cold[v] = Cb[(wi * 32 + 8 * (v / 4) + 4 * h + (v % 4)) * K + wj * 32 + ln];
  }
#pragma unroll
  for (int u = 0; u < NVP; ++u) {
    const int e = (tid + u * NT) * 4, r = e / K, c = e % K;
    float* d = sp + r * kChainLdP + c;
    d[0] = vp[u].x; d[1] = vp[u].y; d[2] = vp[u].z; d[3] = vp[u].w;
  }
  __syncthreads();
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  {
    // X[i][j] = sum_l P[l][i] G[l][j]
    const float* pa = sp + h * kChainLdP + wi * 32 + ln;
#pragma unroll
    for (int t = 0; t < K / 2; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[2 * t * kChainLdP], g[t], acc, 0, 0, 0);
  }
  {
    float* xw = sx + wi * (K * kChainLdX) + (wj * 32 + ln) * kChainLdX;
#pragma unroll
    for (int v = 0; v < 16; ++v) xw[8 * (v / 4) + 4 * h + (v % 4)] = acc[v];
  }
  // (in flight under the second product)
  UpdateOld was[16];
  if (up.T) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      was[v] = update_load(up, size_t(b) * K * K + size_t(wi * 32 + 8 * (v / 4) + 4 * h + (v % 4)) * K + wj * 32 + ln);
  }
  const float denom = up.T && up.denom ? *up.denom : 1.f;
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  {
    // Y[i][j] = sum_l X[i][l] P[j][l]
    const float* pa = sx + wi * (K * kChainLdX) + h * kChainLdX + ln;
    const float* pb = sp + (wj * 32 + ln) * kChainLdP + h;
#pragma unroll 8
    for (int t = 0; t < K / 2; ++t)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[2 * t * kChainLdX], pb[2 * t], acc, 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = wi * 32 + 8 * (v / 4) + 4 * h + (v % 4), j = wj * 32 + ln;
    const float gr = alpha * acc[v] + (beta != 0.f ? beta * cold[v] : 0.f);
    if (up.T) {
      update_store(up, size_t(b) * K * K + size_t(i) * K + j, gr, was[v], denom);
    } else {
      Cb[i * K + j] = gr;
    }
  }
}

// The same for blocks of 128 on the 16-bit matrix pipe: every operand split exactly into three bfloat16 parts, the six part products of
// weight >= 2^-24, float32 accumulation -- six instructions of 32 cycles where eight of 64 do the float32 product.  A workgroup owns 64 rows
// of a block.  It splits its slice of P^T once for all waves (48 KB of LDS, 16-byte operands [part][step of 16][half][row][8]); G's columns are
// split by the wave that multiplies by them, two waves each, and so are P's rows, as they come from memory.  The first product
// is taken as X^T = G^T P: a lane then holds four consecutive contraction indices of the second one, which go to the slice's place in LDS.
// Bound: the splits (880 vector instructions a wave) next to 96 matrix instructions, requests and stores of 4 bytes a lane at both ends
// (72 blocks, 22 k cycles: requests 4, P^T 1.3, first product 4.4, exchange 2, second 8, stores 3; with Adam's state 29 k).
// On v_mfma_f32_32x32x2_f32 / here: 72 blocks 15.7 / 13.2 us, with Adam 20.0 / 18.1, 112 17.4 / 15.2, 288 50 / 37.5.
// Where the whole block of G is below kC16Small its third parts, or X's, would end below bfloat16's smallest number (the gradient of a
// loss in weights of 1e-18 and less is 2^-120): it is taken times 2^60, and alpha divided by it.
constexpr int kC16Part = 8 * 2 * 64 * 16;
constexpr float kC16Small = 0x1p-60f;
__device__ __forceinline__ void split3_pair(float x0, float x1, uint32_t& a, uint32_t& b, uint32_t& c) {
  a = pack_bf16(x0, x1);
  const float r0 = x0 - bf16_lo_f32(a), r1 = x1 - bf16_hi_f32(a);
  b = pack_bf16(r0, r1);
  c = pack_bf16(r0 - bf16_lo_f32(b), r1 - bf16_hi_f32(b));
}
// TWO: two workgroups a compute unit, 128 registers a wave (what the update needs of the old state then comes in two halves).
template <bool TWO>
__global__ __launch_bounds__(512, TWO ? 4 : 2) void bgemm_chain16_kernel(const float* __restrict__ P, const float* __restrict__ G, float* __restrict__ C,
                                                               float alpha, float beta, const UpdateHook up) {
  constexpr int K = 128;
  __shared__ __align__(16) unsigned char op[3 * kC16Part];
  __shared__ float gmax[8];
  int b, slice;
  block_and_part(blockIdx.x, 2, gridDim.x, &b, &slice);
  const int i0 = slice * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), ln = lane & 31, h = lane >> 5;
  const int wi = wave >> 2, wj = wave & 3;
  const float* Pb = P + size_t(b) * K * K;
  const float* Gb = G + size_t(b) * K * K;
  float* Cb = C + size_t(b) * K * K;
  struct Parts { bf16x8 hi, mid, lo; };
  auto split8 = [](const float* x) __attribute__((always_inline)) {
    uintx4 a, m, l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t u, v, w;
      split3_pair(x[2 * i], x[2 * i + 1], u, v, w);
      a[i] = u; m[i] = v; l[i] = w;
    }
    return Parts{as_bf16x8(a), as_bf16x8(m), as_bf16x8(l)};
  };
  auto load3 = [&](int step, int row) __attribute__((always_inline)) {
    const unsigned char* at = op + ((step * 2 + h) * 64 + row) * 16;
    return Parts{as_bf16x8(*reinterpret_cast<const uintx4*>(at)), as_bf16x8(*reinterpret_cast<const uintx4*>(at + kC16Part)),
                 as_bf16x8(*reinterpret_cast<const uintx4*>(at + 2 * kC16Part))};
  };
  auto six = [](const Parts& x, const Parts& y, floatx16 d) __attribute__((always_inline)) {
    d = CAFEQ_MFMA_BF16(x.lo, y.hi, d);
    d = CAFEQ_MFMA_BF16(x.hi, y.lo, d);
    d = CAFEQ_MFMA_BF16(x.mid, y.mid, d);
    d = CAFEQ_MFMA_BF16(x.mid, y.hi, d);
    d = CAFEQ_MFMA_BF16(x.hi, y.mid, d);
    return CAFEQ_MFMA_BF16(x.hi, y.hi, d);
  };
  // the slice of P^T: this thread's row, contraction indices 16 wave .. + 15; and the wave's columns of G
  float v[16], g[64];
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = Pb[(16 * wave + e) * K + i0 + lane];
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) g[8 * s + e] = Gb[(16 * s + 8 * h + e) * K + wj * 32 + ln];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const Parts t = split8(v + 8 * q);
    unsigned char* at = op + ((wave * 2 + q) * 64 + lane) * 16;
    *reinterpret_cast<uintx4*>(at) = __builtin_bit_cast(uintx4, t.hi);
    *reinterpret_cast<uintx4*>(at + kC16Part) = __builtin_bit_cast(uintx4, t.mid);
    *reinterpret_cast<uintx4*>(at + 2 * kC16Part) = __builtin_bit_cast(uintx4, t.lo);
  }
  float gm = 0.f;
#pragma unroll
  for (int e = 0; e < 64; ++e) gm = fmaxf(gm, fabsf(g[e]));
  gm = cluster_allmax<64>(gm);
  if (lane == 0) gmax[wave] = gm;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 8; ++w) gm = fmaxf(gm, gmax[w]);
  if (gm < kC16Small) {                     // (uniform)
    alpha *= kC16Small;
#pragma unroll
    for (int e = 0; e < 64; ++e) g[e] *= 1.f / kC16Small;
  }
  floatx16 x;
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = 0.f;
#pragma unroll
  for (int s = 0; s < 8; ++s) x = six(split8(g + 8 * s), load3(s, wi * 32 + ln), x);
  // rows of P for the second product, half of them ahead of the exchange
  float p[64];
  auto request = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int s = s0; s < s0 + 4; ++s)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float4 t = *reinterpret_cast<const float4*>(Pb + (wj * 32 + ln) * K + 16 * s + 8 * h + 4 * u);
        p[8 * s + 4 * u] = t.x; p[8 * s + 4 * u + 1] = t.y; p[8 * s + 4 * u + 2] = t.z; p[8 * s + 4 * u + 3] = t.w;
      }
  };
  request(0);
  __syncthreads();                          // (the slice of P^T is still being read)
  // X[i = 32 wi + ln][l = 32 wj + 8 q + 4 h + e], e < 4, in register 4 q + e
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t a[2], m[2], l[2];
    split3_pair(x[4 * q], x[4 * q + 1], a[0], m[0], l[0]);
    split3_pair(x[4 * q + 2], x[4 * q + 3], a[1], m[1], l[1]);
    unsigned char* at = op + (((2 * wj + (q >> 1)) * 2 + (q & 1)) * 64 + wi * 32 + ln) * 16 + 8 * h;
    *reinterpret_cast<uint2*>(at) = make_uint2(a[0], a[1]);
    *reinterpret_cast<uint2*>(at + kC16Part) = make_uint2(m[0], m[1]);
    *reinterpret_cast<uint2*>(at + 2 * kC16Part) = make_uint2(l[0], l[1]);
  }
  __syncthreads();
  request(4);
  floatx16 y;
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = 0.f;
#pragma unroll
  for (int s = 0; s < 4; ++s) y = six(load3(s, wi * 32 + ln), split8(p + 8 * s), y);
  constexpr int EB = TWO ? 8 : 16;          // elements of the result whose old state is held at a time
  float cold[EB];
  UpdateOld was[EB];
  auto place = [&](int r) __attribute__((always_inline)) { return (i0 + wi * 32 + 8 * (r / 4) + 4 * h + (r % 4)) * K + wj * 32 + ln; };
  auto old_state = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < EB; ++r) {
      cold[r] = beta != 0.f ? Cb[place(r0 + r)] : 0.f;
      if (up.T) was[r] = update_load(up, size_t(b) * K * K + size_t(place(r0 + r)));
    }
  };
  const float denom = up.T && up.denom ? *up.denom : 1.f;
  // (in flight under the rest of the product)
  if (!TWO) old_state(0);
#pragma unroll
  for (int s = 4; s < 8; ++s) {
    if (TWO && s == 6) old_state(0);
    y = six(load3(s, wi * 32 + ln), split8(p + 8 * s), y);
  }
#pragma unroll
  for (int r0 = 0; r0 < 16; r0 += EB) {
    if (r0 > 0) old_state(r0);
#pragma unroll
    for (int r = 0; r < EB; ++r) {
      const float gr = alpha * y[r0 + r] + (beta != 0.f ? beta * cold[r] : 0.f);
      if (up.T) update_store(up, size_t(b) * K * K + size_t(place(r0 + r)), gr, was[r], denom);
      else Cb[place(r0 + r)] = gr;
    }
  }
}

// Blocks of 32, a workgroup per block: (P^T G) P^T, X = P^T G in LDS (two launches with X in memory before: 45 blocks 4.7 + 4.1 us).  A thread
// takes four neighbouring elements of a row, so that a step of either sum is one broadcast and one 16-byte read for four
// multiply-adds (an element at a time, eight reads for them: the launch below 9.8 us at 8 blocks and 11.4 at 90, now 5.5 and 6.5).
constexpr int kC32Ld = 36;                  // floats a row (16-byte vectors; eight rows of a wave in different banks)
struct Chain32Lds {
  float p[32 * kC32Ld], pt[32 * kC32Ld], g[32 * kC32Ld], x[32 * kC32Ld];   // P, P^T, G, X
};
// the thread's four elements of P (row tid / 8, columns 4 (tid % 8) ..) into both orders
__device__ __forceinline__ void chain32_put(Chain32Lds& s, const float4 p) {
  const int i = int(threadIdx.x) >> 3, j = 4 * (int(threadIdx.x) & 7);
  *reinterpret_cast<float4*>(s.p + i * kC32Ld + j) = p;
  s.pt[j * kC32Ld + i] = p.x; s.pt[(j + 1) * kC32Ld + i] = p.y; s.pt[(j + 2) * kC32Ld + i] = p.z; s.pt[(j + 3) * kC32Ld + i] = p.w;
}
// P, P^T and G are in LDS, behind a barrier: the thread's four elements of the product
__device__ __forceinline__ float4 chain32(Chain32Lds& s) {
  const int i = int(threadIdx.x) >> 3, j = 4 * (int(threadIdx.x) & 7);
  auto product = [&](const float* a, int sa, const float* b) __attribute__((always_inline)) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int l = 0; l < 32; ++l) {
      const float x = a[l * sa];
      const float4 y = *reinterpret_cast<const float4*>(b + l * kC32Ld);
      acc.x = fmaf(x, y.x, acc.x); acc.y = fmaf(x, y.y, acc.y); acc.z = fmaf(x, y.z, acc.z); acc.w = fmaf(x, y.w, acc.w);
    }
    return acc;
  };
  *reinterpret_cast<float4*>(s.x + i * kC32Ld + j) = product(s.p + i, kC32Ld, s.g + j);   // X[i][j] = sum_l P[l][i] G[l][j]
  __syncthreads();
  return product(s.x + i * kC32Ld, 1, s.pt + j);                                         // Y[i][j] = sum_l X[i][l] P[j][l]
}
struct UpdateOld4 { float4 t, m, v; };
__device__ __forceinline__ UpdateOld4 update_load4(const UpdateHook& u, size_t at) {
  UpdateOld4 o{};
  if (u.T) {
    o.t = *reinterpret_cast<const float4*>(u.T + at);
    if (u.m) { o.m = *reinterpret_cast<const float4*>(u.m + at); o.v = *reinterpret_cast<const float4*>(u.v + at); }
  }
  return o;
}
__device__ __forceinline__ void update_store4(const UpdateHook& u, size_t at, float4 g, const UpdateOld4& o, float denom) {
  update_store(u, at, g.x, UpdateOld{o.t.x, o.m.x, o.v.x}, denom);
  update_store(u, at + 1, g.y, UpdateOld{o.t.y, o.m.y, o.v.y}, denom);
  update_store(u, at + 2, g.z, UpdateOld{o.t.z, o.m.z, o.v.z}, denom);
  update_store(u, at + 3, g.w, UpdateOld{o.t.w, o.m.w, o.v.w}, denom);
}
// C = beta C + alpha (P^T G) P^T
__global__ __launch_bounds__(256) void bgemm_chain32_kernel(const float* __restrict__ P, const float* __restrict__ G,
                                                            float* __restrict__ C, float alpha, float beta,
                                                            const UpdateHook up) {
  __shared__ __align__(16) Chain32Lds s;
  const size_t at = size_t(blockIdx.x) * 1024 + 4 * threadIdx.x;
  const float4 p = *reinterpret_cast<const float4*>(P + at), g = *reinterpret_cast<const float4*>(G + at);
  const float4 cold = beta != 0.f ? *reinterpret_cast<const float4*>(C + at) : make_float4(0.f, 0.f, 0.f, 0.f);
  const UpdateOld4 old = update_load4(up, at);
  const float denom = up.T && up.denom ? *up.denom : 1.f;
  chain32_put(s, p);
  *reinterpret_cast<float4*>(s.g + (threadIdx.x >> 3) * kC32Ld + 4 * (threadIdx.x & 7)) = g;
  __syncthreads();
  const float4 y = chain32(s);
  const float4 r = beta != 0.f ? make_float4(alpha * y.x + beta * cold.x, alpha * y.y + beta * cold.y, alpha * y.z + beta * cold.z,
                                             alpha * y.w + beta * cold.w)
                               : make_float4(alpha * y.x, alpha * y.y, alpha * y.z, alpha * y.w);
  if (up.T) update_store4(up, at, r, old, denom);
  else *reinterpret_cast<float4*>(C + at) = r;
}

// What follows the loss / gradient kernel of a single matrix with blocks of 32, in one launch: a workgroup per block sums its
// partials, forms the middle factor and adds its way through the inverse (the work of single_tail_kernel and
// bgemm_chain32_kernel, sums in their order, nothing of it through memory in between); one more workgroup reduces the losses.
// A gradient-descent step that divides by ||W||^2 sums it from the headers itself, in that workgroup's order.
// Bound: the latencies of headers and partials, each with eight requests in flight: 5.5 us at
// 8 blocks, 6.5 at 90, against 4.0 + 5.7 and 4.9 + 5.7 in two launches.
// INV: a learning loop's step, with the inverse of the transform it leaves (warm-started from P, in P's place) by the first wave: what a
// launch of its own took for itself and its loads (1147 x 2880, eight steps 208 -> 195 us).
template <bool INV>
__global__ __launch_bounds__(256) void tail_chain32_kernel(const ReduceArgs ra, const VArgs va, const LossArgs la, const float* P,
                                                           const UpdateHook up, float* Tinv, int* status) {
  constexpr int K = 32;
  __shared__ __align__(16) Chain32Lds s;
  __shared__ __align__(16) float v[K];
  __shared__ double red[5 * (kLossThreads / 64)];
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    double m, sm;
    reduce_losses_body<kLossThreads>(la, red, true, &m, &sm);
    return;
  }
  const int b = int(blockIdx.x) - 1, i = tid >> 3, j = 4 * (tid & 7);
  const size_t at = size_t(b) * K * K + 4 * tid;
  const float4 p = *reinterpret_cast<const float4*>(P + at);
  const UpdateOld4 old = update_load4(up, at);
  double wsq = 0;
  if (up.denom) {
    float t[4];
    for (int k0 = tid; k0 < la.nslotA; k0 += 4 * kLossThreads) {
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = k0 + u * kLossThreads < la.nslotA ? la.hdrA[size_t(k0 + u * kLossThreads) * kHdrFloats + kHdrWsq] : 0.f;
#pragma unroll
      for (int u = 0; u < 4; ++u) wsq += t[u];
    }
  }
  // the middle factor's v: thread n (of every 32 the same) index n, the headers' order
  double vn = 0;
  for (int q = b * va.rep; q < (b + 1) * va.rep; ++q) {
    // (segments and groups of 32 to 256: powers of two)
    const int64_t ax = int64_t(q) * K + tid % K, seg = ax >> __builtin_ctz(va.L);
    const float* h0 = va.slot_hdr + seg * kHdrFloats + kHdrVa2 + ((int(ax) & (va.L - 1)) >> __builtin_ctz(va.G));
    int lo, hi;
    seg_wg_range(seg, va.mt_per_seg, va.n_mt, va.nwg, &lo, &hi);
    for (int w0 = lo; w0 < hi; w0 += 8) {
      float t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = w0 + u < hi ? h0[int64_t(w0 + u) * kHdrFloats] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) vn += t[u];
    }
  }
  // the gradient's partials: four inputs of output row i
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int q = b * ra.rep; q < (b + 1) * ra.rep; ++q) {
    const int64_t ax = int64_t(q) * K, seg = ax >> __builtin_ctz(ra.seg_len);
    const float* part = ra.slot_grad + seg * ra.part_floats + (int(ax) & (ra.seg_len - 1)) * K + 4 * tid;
    int lo, hi;
    seg_wg_range(seg, ra.mt_per_seg, ra.n_mt, ra.nwg, &lo, &hi);
    for (int w0 = lo; w0 < hi; w0 += 8) {
      float4 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        t[u] = w0 + u < hi ? *reinterpret_cast<const float4*>(part + int64_t(w0 + u) * ra.part_floats) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 8; ++u) { acc.x += t[u].x; acc.y += t[u].y; acc.z += t[u].z; acc.w += t[u].w; }
    }
  }
  if (tid < K) v[tid] = float(vn * va.beta);
  chain32_put(s, p);
  if (up.denom) {
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) wsq += __shfl_xor(wsq, k);
    if ((tid & 63) == 0) red[tid >> 6] = wsq;
  }
  __syncthreads();
  {
    float4 g = p;
    if (va.scale_rows) {
      const float f = v[i];
      g.x *= f; g.y *= f; g.z *= f; g.w *= f;
    } else {
      const float4 f = *reinterpret_cast<const float4*>(v + j);
      g.x *= f.x; g.y *= f.y; g.z *= f.z; g.w *= f.w;
    }
    *reinterpret_cast<float4*>(s.g + i * kC32Ld + j) = g;
  }
  __syncthreads();
  const float4 y = chain32(s);
  if (ra.transpose_out) {
    // out[m][j] = acc[j][m]: through G's room, which the first product is done with
    s.g[j * kC32Ld + i] = acc.x; s.g[(j + 1) * kC32Ld + i] = acc.y; s.g[(j + 2) * kC32Ld + i] = acc.z; s.g[(j + 3) * kC32Ld + i] = acc.w;
    __syncthreads();
    acc = *reinterpret_cast<const float4*>(s.g + i * kC32Ld + j);
  }
  const float4 r = make_float4(-2.f * y.x + acc.x, -2.f * y.y + acc.y, -2.f * y.z + acc.z, -2.f * y.w + acc.w);
  float denom = 1.f;
  if (up.denom) {
    double t = 0;
    for (int k = 0; k < kLossThreads / 64; ++k) t += red[k];
    denom = float(t);
  }
  if (up.T) update_store4(up, at, r, old, denom);
  else *reinterpret_cast<float4*>(ra.out + at) = r;
  if constexpr (INV) {
    static_assert(NsShape<K>::bytes <= sizeof(Chain32Lds) && NsShape<K>::NW == 1, "one wave, in the chain's room");
    __syncthreads();                                  // (the block's new entries are written, the chain's LDS is free)
    if (tid >= 64) return;
    if (!ns_inverse_body<K, 1>(up.T, Tinv, status, b, reinterpret_cast<unsigned char*>(&s)))
      gj_panel_body<K, 4, 4, double, true>(ns_eliminate_args(K, up.T, Tinv, status), b, *reinterpret_cast<GjShared<K, double>*>(&s));
  }
}

// K == 32: one 32 x 32 product per workgroup, C = alpha A B + beta C
__global__ __launch_bounds__(256) void bgemm32_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                       float* __restrict__ C, float alpha, float beta) {
  constexpr int K = 32;
  __shared__ float sa[K][K + 1], sb[K][K + 1];
  const float* Ab = A + size_t(blockIdx.x) * K * K;
  const float* Bb = B + size_t(blockIdx.x) * K * K;
  float* Cb = C + size_t(blockIdx.x) * K * K;
  for (int e = threadIdx.x; e < K * K; e += 256) {
    sa[e / K][e % K] = Ab[e];
    sb[e / K][e % K] = Bb[e];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < K * K; e += 256) {
    const int i = e / K, j = e % K;
    float acc = 0.f;
#pragma unroll
    for (int l = 0; l < K; ++l) acc = fmaf(sa[i][l], sb[l][j], acc);
    Cb[e] = alpha * acc + (beta != 0.f ? beta * Cb[e] : 0.f);
  }
}

}  // namespace

// Whether a rho request can also form the group sums of rho_group_kernel for groups of G axis indices.
bool rho_groups_inline(int K, int nb, int G, int rep) {
  if (G >= 1 && G <= K) return K % G == 0;
  return rep == 1 && G <= 256 && G % K == 0 && nb % (G / K) == 0;
}
int launch_split_planes_multi(const SplitRequest* req, int n, int K, int nb, hipStream_t st, float* hdr,
                              int64_t nslot, const RhoRequest* rho, int nrho) {
  if (n > 4 || nrho > 2) return CAFEQ_ERR_INVALID_ARG;
  SplitJobs js;
  js.njobs = n; js.nrho = nrho; js.nb = nb; js.hdr = hdr; js.nhdr = nslot * kHdrFloats;
  for (int i = 0; i < n; ++i) {
    js.job[i].src = req[i].src; js.job[i].dst = req[i].dst;
    js.job[i].trans = req[i].trans; js.job[i].nplanes = req[i].nplanes;
    js.job[i].fscale = req[i].fscale; js.job[i].natural = req[i].natural; js.job[i].texp = req[i].texp;
    js.job[i].minus_one = req[i].minus_one;
  }
  for (int i = 0; i < nrho; ++i) {
    if (rho[i].rG && !rho_groups_inline(K, nb, rho[i].G, rho[i].rep)) return CAFEQ_ERR_INVALID_ARG;
    js.rho[i] = RhoJob{rho[i].P, rho[i].rho, rho[i].rG, rho[i].by_row, rho[i].G, rho[i].rep,
                       rho[i].rG && rho[i].G > K ? rho[i].G / K : 1};
  }
  // one workgroup per (block, job) when those fill the chip; else one per (block, job, stage)
  const dim3 grid(nb, n + nrho, n == 0 || (K < 256 && nb * n >= 128) ? 1 : K / 32);
  switch (K) {
    case 32: hipLaunchKernelGGL(split_planes_kernel<32>, grid, dim3(kSplitThreads), 0, st, js); break;
    case 64: hipLaunchKernelGGL(split_planes_kernel<64>, grid, dim3(kSplitThreads), 0, st, js); break;
    case 128: hipLaunchKernelGGL(split_planes_kernel<128>, grid, dim3(kSplitThreads), 0, st, js); break;
    case 256: hipLaunchKernelGGL(split_planes_kernel<256>, grid, dim3(kSplitThreads), 0, st, js); break;
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
int launch_rho_groups(const float* rho, int K, int rep, int G, int64_t ngroups, float* rG, hipStream_t st) {
  const int wpg = G >= 1024 ? kRhoGroupWaves : 1, per = kRhoGroupWaves / wpg;
  hipLaunchKernelGGL(rho_group_kernel, dim3(unsigned((ngroups + per - 1) / per)), dim3(kRhoGroupWaves * kWave), 0, st, rho,
                     31 - __builtin_clz(unsigned(K)), rep, G, ngroups, wpg, rG);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
namespace {
// fused: the partials were written by the fused kernel (segments of max(K, G), [NBLK][K][K]); otherwise by the
// gradient pass (chunks of 128 inputs; halves of the inputs for K == 256)
ReduceArgs reduce_args(const CoreParams& p, int K, int G, bool fused, int transpose_out, const double* lse_ms,
                       const float* member_ref, float* out) {
  ReduceArgs a;
  a.slot_grad = p.slot_grad; a.slot_hdr = p.slot_hdr; a.mt_per_seg = p.mt_per_seg; a.n_mt = p.n_mt;
  a.nwg = p.nwg; a.nseg = p.nseg; a.K = K; a.rep = p.rep;
  if (fused) {
    const int L = K > G ? K : G;
    a.seg_len = L; a.part_floats = L * K; a.msplit = 1;
  } else {
    a.seg_len = 128; a.msplit = K == 256 ? 2 : 1; a.part_floats = K == 256 ? 256 * 128 : 128 * K;
  }
  a.transpose_out = transpose_out; a.t = p.lse_t; a.lse_ms = lse_ms; a.member_ref = member_ref; a.out = out;
  return a;
}
}  // namespace
int launch_reduce_grad(const CoreParams& p, int K, int G, bool fused, int nb, int transpose_out,
                       const double* lse_ms, const float* member_ref, float* out, hipStream_t st) {
  ReduceJobs js;
  js.job[0] = js.job[1] = reduce_args(p, K, G, fused, transpose_out, lse_ms, member_ref, out);
  hipLaunchKernelGGL(reduce_grad_kernel, dim3(nb, (K * K + 1023) / 1024, 1), dim3(256), 0, st, js);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
// Both members of a pair in one launch: pa -> outA (transposed), pb -> outB.
int launch_reduce_grad_pair(const CoreParams& pa, int GA, bool fusedA, const float* refA, float* outA,
                            const CoreParams& pb, int GB, bool fusedB, const float* refB, float* outB, int K,
                            int nb, const double* lse_ms, hipStream_t st) {
  ReduceJobs js;
  js.job[0] = reduce_args(pa, K, GA, fusedA, 1, lse_ms, refA, outA);
  js.job[1] = reduce_args(pb, K, GB, fusedB, 0, lse_ms, refB, outB);
  hipLaunchKernelGGL(reduce_grad_kernel, dim3(nb, (K * K + 1023) / 1024, 2), dim3(256), 0, st, js);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
int launch_build_mmid(const CoreParams& p, int K, int G, int nb, const float* P, int scale_rows, float* Mmid,
                      hipStream_t st) {
  const VArgs a = mmid_args(p, K, K > G ? K : G, G, P, scale_rows, Mmid);
  hipLaunchKernelGGL(build_mmid_kernel, dim3(nb * kMmidParts), dim3(256), 0, st, a);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
int launch_single_tail(const CoreParams& pgrad, const CoreParams& ploss, int K, int G, bool fused, int nb,
                       int transpose_out, float* gradT, const float* P, int scale_rows, float* Mmid, float beta,
                       int nslot, float* losses, double* lse_ms, hipStream_t st) {
  const ReduceArgs ra = reduce_args(pgrad, K, G, fused, transpose_out, nullptr, nullptr, gradT);
  const VArgs va = mmid_args(ploss, K, K > G ? K : G, G, P, scale_rows, Mmid);
  LossArgs la{};
  la.hdrA = ploss.slot_hdr; la.nslotA = nslot; la.kind = kLossSur; la.beta = beta; la.losses = losses;
  la.lse_ms = lse_ms;
  const int nred_x = nb, nred_y = (K * K + 1023) / 1024;
  hipLaunchKernelGGL(single_tail_kernel, dim3(unsigned(nred_x * nred_y + nb * kMmidParts + 1)), dim3(256), 0, st, ra, va, la,
                     nred_x, nred_y, nb);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
// the same with the gradient's way through the inverse and the update (blocks of 32; hook->denom, if any: losses[2])
int launch_tail_chain32(const CoreParams& pgrad, const CoreParams& ploss, int G, bool fused, int nb, int transpose_out, float* gradT,
                        const float* P, int scale_rows, float beta, int nslot, float* losses, double* lse_ms, hipStream_t st,
                        const UpdateHook* hook, float* Tinv, int* status) {
  constexpr int K = 32;
  if (Tinv && !(hook && hook->T)) return CAFEQ_ERR_INVALID_ARG;
  if (hook && hook->denom && hook->denom != losses + 2) return CAFEQ_ERR_INVALID_ARG;
  const ReduceArgs ra = reduce_args(pgrad, K, G, fused, transpose_out, nullptr, nullptr, gradT);
  const VArgs va = mmid_args(ploss, K, K > G ? K : G, G, P, scale_rows, nullptr);
  LossArgs la{};
  la.hdrA = ploss.slot_hdr; la.nslotA = nslot; la.kind = kLossSur; la.beta = beta; la.losses = losses;
  la.lse_ms = lse_ms;
  const UpdateHook up = hook ? *hook : UpdateHook{};
  if (Tinv) hipLaunchKernelGGL(tail_chain32_kernel<true>, dim3(unsigned(nb + 1)), dim3(256), 0, st, ra, va, la, P, up, Tinv, status);
  else hipLaunchKernelGGL(tail_chain32_kernel<false>, dim3(unsigned(nb + 1)), dim3(256), 0, st, ra, va, la, P, up, Tinv, status);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
int launch_reduce_losses(int kind, const float* hdrA, int nslotA, const float* hdrB, int nslotB, float beta,
                         float t, int64_t ngroups, float* losses, double* lse_ms, hipStream_t st) {
  LossArgs a;
  a.hdrA = hdrA; a.nslotA = nslotA; a.hdrB = hdrB; a.nslotB = nslotB; a.kind = kind; a.beta = beta; a.t = t;
  a.ngroups = ngroups; a.losses = losses; a.lse_ms = lse_ms;
  hipLaunchKernelGGL(reduce_losses_kernel, dim3(1), dim3(kLossThreads), 0, st, a);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
// Transposed operands for blocks of 256 alone (the smaller blocks' chains take both products in one launch).
int launch_bgemm(bool ta, bool tb, const float* A, const float* B, float* C, int K, int nb, float alpha,
                 float beta, hipStream_t st, const UpdateHook* hook) {
  const UpdateHook up = hook ? *hook : UpdateHook{};
  if ((ta && tb) || ((ta || tb) && K != 256) || (hook && K == 32)) return CAFEQ_ERR_INVALID_ARG;
  const unsigned grid = unsigned(nb) * (K / 64) * (K / 64);
  if (K == 32) {
    hipLaunchKernelGGL(bgemm32_kernel, dim3(nb), dim3(256), 0, st, A, B, C, alpha, beta);
  } else if (K == 64) {
    hipLaunchKernelGGL((bgemm_mfma_kernel<false, false, 64>), dim3(grid), dim3(256), 2 * 64 * 65 * sizeof(float), st, A, B, C, K,
                       alpha, beta, up);
  } else {
    constexpr int CH = 128;
    constexpr size_t lds = 2 * CH * 65 * sizeof(float);
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
      bool ok = true;
#define CAFEQ_ATTR(TA, TB)                                                                                     \
  ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(bgemm_mfma_kernel<TA, TB, CH>),                 \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) == hipSuccess
      CAFEQ_ATTR(true, false); CAFEQ_ATTR(false, true); CAFEQ_ATTR(false, false);
#undef CAFEQ_ATTR
#define CAFEQ_ATTR(TA, TB)                                                                                        \
  ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(bgemm_mfma_kernel<TA, TB, CH, 2>),                 \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(2 * lds)) == hipSuccess
      CAFEQ_ATTR(true, false);
#undef CAFEQ_ATTR
      if (!ok) return CAFEQ_ERR_LAUNCH;
      attr_set = true;
    }
#define CAFEQ_G128(TA, TB) hipLaunchKernelGGL((bgemm_mfma_kernel<TA, TB, CH>), dim3(grid), dim3(256), lds, st, A, B, C, K, alpha, beta, up)
    // (transposed: K = 256)
    if (ta && int64_t(grid) <= device_cu_count()) {
      hipLaunchKernelGGL((bgemm_mfma_kernel<true, false, CH, 2>), dim3(grid), dim3(512), 2 * lds, st, A, B, C, K, alpha, beta, up);
    } else if (ta) {
      CAFEQ_G128(true, false);
    } else if (tb) {
      CAFEQ_G128(false, true);
    } else {
      CAFEQ_G128(false, false);
    }
#undef CAFEQ_G128
  }
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
// C = beta C + alpha P^T G P^T per block; x1: scratch of nb K K floats for blocks of 256
int launch_bgemm_chain(const float* P, const float* G, float* x1, float* C, int K, int nb, float alpha, float beta,
                       hipStream_t st, const UpdateHook* hook) {
  if (K == 256) {
    const int rc = launch_bgemm(true, false, P, G, x1, K, nb, 1.f, 0.f, st);
    if (rc) return rc;
    return launch_bgemm(false, true, x1, P, C, K, nb, alpha, beta, st, hook);
  }
  const UpdateHook up = hook ? *hook : UpdateHook{};
  switch (K) {
    case 32: hipLaunchKernelGGL(bgemm_chain32_kernel, dim3(unsigned(nb)), dim3(256), 0, st, P, G, C, alpha, beta, up); break;
    case 64:
      hipLaunchKernelGGL(bgemm_chain64_kernel, dim3(unsigned(nb)), dim3(256), kChain64Lds, st, P, G, C, alpha, beta, up);
      break;
    case 128:
      // more workgroups than compute units: the form of which two fit one
      if (2 * int64_t(nb) > device_cu_count())
        hipLaunchKernelGGL(bgemm_chain16_kernel<true>, dim3(unsigned(nb) * 2), dim3(512), 0, st, P, G, C, alpha, beta, up);
      else
        hipLaunchKernelGGL(bgemm_chain16_kernel<false>, dim3(unsigned(nb) * 2), dim3(512), 0, st, P, G, C, alpha, beta, up);
      break;
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
int device_cu_count() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cus = n;
  }
  return cus;
}

}  // namespace cafeq
