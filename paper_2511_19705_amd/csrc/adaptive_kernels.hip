// Kernels of the adaptive-rounding step (paper Sec. 5, Alg. 1) in transformed coordinates.
//
// Alg. 1 alternates  W2^ <- Q(pinv(W1^) W1 W2)  and  W1^ <- Q(W1 W2 pinv(W2^)).  Per head the
// pseudoinverse of a full-column-rank (resp. full-row-rank) quantized block is formed from
// k x k normal equations.  With Xq the dequantized codes and E = Xq - X the current rounding
// error, both lines have the same shape:
//     S = Gram(Xq, Xq),  R = Gram(Xq, E),   C = I - S^-1 R
// where Gram(X, Y)[a][b] = sum_t X[t][a] Y[t][b]; t runs over the rows of U (line 3) or over
// the columns of the head's row-blocks of V (line 4), a and b over the k indices of the head.
// Line 3 quantizes C . V_q, line 4 quantizes U_b . C^T (the fused core is handed C as the
// [out][in] operand either way).  Working with E instead of X keeps the float32 Gram sums at
// the scale of the correction, not of the identity it is subtracted from.
//
//   gram_pair_kernel : fp32 MFMA (v_mfma_f32_32x32x2_f32), one workgroup per (head, 32-row
//                      output stripe, chunk of the contraction range); codes are dequantized
//                      on the fly; chunk partials are written out, not atomically added.
//   gram_pair16_kernel : the same pair for heads of 128 and 256 on the 16-bit matrix pipe, operands
//                      split exactly into three bfloat16 parts (groups of 32);
//   gram_pair_codes_kernel : with the codes themselves on one side (longer groups).
//   gj_panel_kernel  : (gj_panel.hpp) sums the chunk partials of S in float64 and inverts it by register-
//                      resident Gauss-Jordan elimination.  C = I - S^-1 R follows as a batched product.
//   gj_spd256_kernel : the inversion of S for heads of 256 as a block elimination whose products
//                      run on the 16-bit matrix pipe.
#include <atomic>

#include "gj_panel.hpp"

namespace cafeq {

namespace {

struct GramArgs {
  const float* X;        // original (transformed) matrix, float32 dense
  const int8_t* codes;   // its current codes
  const float* scales;   // its current scales
  int64_t rows, cols;
  int K, G, rep;
  int64_t tlen;          // contraction length per row-block (rows of U / columns of V)
  int64_t chunk;         // contraction elements per workgroup (multiple of 16)
  int nchunk;            // chunks per row-block
  float* partial;        // [nb][rep*nchunk][2 or 3][K][K]: Gram(Xq,Xq), Gram(Xq,E) and, TRIPLE, Gram(E,E)
};

// AXIS == COL: t = row i, free index = column;  AXIS == ROW: t = column c, free index = row.
// One workgroup per (head, 32-row output stripe jt1, chunk of the contraction range).  Per step
// of 16 contraction indices the workgroup loads the head's 16 x K slab of codes, scales and
// originals with wide coalesced loads, dequantizes it ONCE (Xq and E = Xq - X) into LDS laid out
// [t][free index], and every wave feeds its MFMAs from there: A = Xq[t][stripe columns] (shared
// by the waves), B = Xq / E [t][its output tiles].  The next slab's loads are in flight while
// the matrix cores work on the current one.
template <int AXIS, int K, bool TRIPLE>
__global__ __launch_bounds__(256) void gram_pair_kernel(const GramArgs a) {
  // row stride of the LDS slab: 16-byte aligned rows for the vector stores of the column case;
  // K + 2 for the row case, whose transposing scalar stores then spread over all banks
  constexpr int KT = K / 32, LD = AXIS == CAFEQ_AXIS_COL ? K + 4 : K + 2;
  __shared__ __align__(16) float qs[16 * LD];
  __shared__ __align__(16) float es[16 * LD];
  const int b = blockIdx.x, jt1 = blockIdx.y;
  const int z = blockIdx.z;                      // (row-block within head, chunk)
  const int qi = z / a.nchunk, ch = z % a.nchunk;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 31, h = lane >> 5;
  const int64_t t0 = int64_t(ch) * a.chunk;
  const int64_t t1 = t0 + a.chunk < a.tlen ? t0 + a.chunk : a.tlen;
  // free-index origin of this head / row-block
  const int64_t f0 = AXIS == CAFEQ_AXIS_COL ? int64_t(b) * K : (int64_t(b) * a.rep + qi) * K;
  const int64_t C = a.cols;

  // output tiles of this wave: jt2 = wave + 4u, u < NU; for K < 128 the waves beyond KT have none.  NU is a
  // compile-time count so that the accumulators stay where the matrix instructions want them.
  constexpr int NU = (KT + 3) / 4;
  const bool active = KT >= 4 || wave < KT;   // known at compile time for K >= 128: no branch around the MFMAs
  floatx16 accS[NU], accR[NU], accT[TRIPLE ? NU : 1];
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int v = 0; v < 16; ++v) { accS[u][v] = 0.f; accR[u][v] = 0.f; accT[TRIPLE ? u : 0][v] = 0.f; }

  // ---- loader roles.  COL: thread -> (t = l / (K/EPT), EPT/4 chunks of four columns, the chunks of the
  // K/EPT threads of a row interleaved so that their 16-byte LDS stores fall into distinct banks);
  // ROW: NP passes of 64 rows, thread -> (row = pass*64 + l/4, four consecutive t = 4*(l%4) ..)
  constexpr int EPT = K >= 64 ? K / 16 : 4;          // COL: columns per thread
  constexpr int NLD = 16 * K / EPT;                  // COL: active loader threads
  constexpr int NP = (K + 63) / 64;                  // ROW: passes
  uint32_t rc[AXIS == CAFEQ_AXIS_COL ? EPT / 4 : NP];
  float4 rx[AXIS == CAFEQ_AXIS_COL ? EPT / 4 : NP];
  float4 rs[AXIS == CAFEQ_AXIS_COL ? EPT / 4 : NP];  // COL: .x only, one scale per chunk
  constexpr int TPR = K / EPT;                       // COL: threads per slab row; chunk j starts at column 4 (l % TPR) + 4 TPR j
  bool rok[AXIS == CAFEQ_AXIS_COL ? 1 : NP];

  auto issue = [&](int64_t t) {
    if (AXIS == CAFEQ_AXIS_COL) {
      const int tt = tid / TPR, c0 = (tid % TPR) * 4;
      const int64_t i = t + tt;
      rok[0] = tid < NLD && i < t1;
      if (rok[0]) {
#pragma unroll
        for (int j = 0; j < EPT / 4; ++j) {
          const int64_t col = f0 + c0 + 4 * TPR * j;
          rs[j].x = a.scales[i * (C / a.G) + col / a.G];
          rc[j] = *reinterpret_cast<const uint32_t*>(a.codes + i * C + col);
          rx[j] = *reinterpret_cast<const float4*>(a.X + i * C + col);
        }
      }
    } else {
#pragma unroll
      for (int pz = 0; pz < NP; ++pz) {
        const int r = pz * 64 + tid / 4;
        const int64_t c = t + 4 * (tid % 4);
        rok[pz] = r < K && c < t1;                  // tlen and chunk are multiples of 4
        if (rok[pz]) {
          const int64_t row = f0 + r;
          rs[pz] = *reinterpret_cast<const float4*>(a.scales + (row / a.G) * C + c);
          rc[pz] = *reinterpret_cast<const uint32_t*>(a.codes + row * C + c);
          rx[pz] = *reinterpret_cast<const float4*>(a.X + row * C + c);
        }
      }
    }
  };
  auto commit = [&]() {
    if (AXIS == CAFEQ_AXIS_COL) {
      if (tid < NLD) {
        const int tt = tid / TPR, c0 = (tid % TPR) * 4;
#pragma unroll
        for (int j = 0; j < EPT / 4; ++j) {
          float4 q = make_float4(0.f, 0.f, 0.f, 0.f), e = q;
          if (rok[0]) {
            const uint32_t cw = rc[j];
            q.x = __fmul_rn(float(int8_t(cw)), rs[j].x);
            q.y = __fmul_rn(float(int8_t(cw >> 8)), rs[j].x);
            q.z = __fmul_rn(float(int8_t(cw >> 16)), rs[j].x);
            q.w = __fmul_rn(float(int8_t(cw >> 24)), rs[j].x);
            e = make_float4(q.x - rx[j].x, q.y - rx[j].y, q.z - rx[j].z, q.w - rx[j].w);
          }
          *reinterpret_cast<float4*>(qs + tt * LD + c0 + 4 * TPR * j) = q;
          *reinterpret_cast<float4*>(es + tt * LD + c0 + 4 * TPR * j) = e;
        }
      }
    } else {
#pragma unroll
      for (int pz = 0; pz < NP; ++pz) {
        const int r = pz * 64 + tid / 4, tq = 4 * (tid % 4);
        if (r < K) {
          float q[4] = {0.f, 0.f, 0.f, 0.f}, e[4] = {0.f, 0.f, 0.f, 0.f};
          if (rok[pz]) {
            const uint32_t cw = rc[pz];
            q[0] = __fmul_rn(float(int8_t(cw)), rs[pz].x);
            q[1] = __fmul_rn(float(int8_t(cw >> 8)), rs[pz].y);
            q[2] = __fmul_rn(float(int8_t(cw >> 16)), rs[pz].z);
            q[3] = __fmul_rn(float(int8_t(cw >> 24)), rs[pz].w);
            e[0] = q[0] - rx[pz].x; e[1] = q[1] - rx[pz].y; e[2] = q[2] - rx[pz].z; e[3] = q[3] - rx[pz].w;
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            qs[(tq + j) * LD + r] = q[j];
            es[(tq + j) * LD + r] = e[j];
          }
        }
      }
    }
  };

  issue(t0);
  for (int64_t t = t0; t < t1; t += 16) {
    commit();
    __syncthreads();
    if (t + 16 < t1) issue(t + 16);
    if (active) {
      const float* pa = qs + h * LD + jt1 * 32 + ln;
      const float* pe = es + h * LD + jt1 * 32 + ln;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float xa = pa[2 * e * LD];
        const float ea = TRIPLE ? pe[2 * e * LD] : 0.f;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          const int off = (2 * e + h) * LD + (wave + 4 * u) * 32 + ln;
          accS[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa, qs[off], accS[u], 0, 0, 0);
          accR[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa, es[off], accR[u], 0, 0, 0);
          if (TRIPLE) accT[TRIPLE ? u : 0] = __builtin_amdgcn_mfma_f32_32x32x2f32(ea, es[off], accT[TRIPLE ? u : 0], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }

  // partial[b][z][0|1(|2)][row][col]
  float* out = a.partial + ((size_t(b) * gridDim.z + z) * (TRIPLE ? 3 : 2)) * size_t(K) * K;
  if (active)
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int col = (wave + 4 * u) * 32 + ln;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = jt1 * 32 + 8 * (v / 4) + 4 * h + (v % 4);
        out[size_t(row) * K + col] = accS[u][v];
        out[size_t(K) * K + size_t(row) * K + col] = accR[u][v];
        if (TRIPLE) out[2 * size_t(K) * K + size_t(row) * K + col] = accT[TRIPLE ? u : 0][v];
      }
    }
}

// The same pair of Gram matrices for heads of 128 and 256 on the 16-bit matrix pipe.  Every float32 value -- the
// dequantized code Xq = fl(q s) and the error E = fl(Xq - X), the numbers the kernel above multiplies -- is split
// exactly into three bfloat16 parts (8 + 8 + 8 significant bits) and a product keeps the six part products of
// weight >= 2^-24 (hh, hm, mh, hl, lh, mm), float32 accumulation: the accuracy of the float32 instruction at 6/16 of
// its time.  So that the split is not repeated per 32-row stripe, a workgroup of eight waves owns a whole 128 x 128
// quadrant of a head's outputs (grid y: quadrant; 1 or 4 per head): per step of 16 contraction indices its 512
// threads each take eight consecutive contraction indices of one free index -- waves 0-3 the quadrant's row side
// (Xq), waves 4-7 its column side (Xq and E) -- dequantize, split, and store one 16-byte matrix-instruction operand
// per part into LDS ([part][half of the step][free index][8 contraction indices], two buffers, one barrier per step); then wave w
// accumulates the tiles (row tile w / 2; column tiles 2 (w % 2), 2 (w % 2) + 1) of S and R: 24 matrix instructions
// from 15 operand reads.  Partials in the layout of the kernel above.
constexpr int kG16PlaneB = 128 * 32;                 // one part of one side: 2 halves x 128 free indices x 8 bfloat16
constexpr int kG16BufB = 9 * kG16PlaneB;             // row side Xq, column side Xq, column side E: 3 parts each
constexpr size_t kG16Lds = 2 * kG16BufB;

__device__ __forceinline__ void split3_bf16(const float (&x)[8], uintx4& ph, uintx4& pm, uintx4& pl) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float x0 = x[2 * i], x1 = x[2 * i + 1];
    const uint32_t h = pack_bf16(x0, x1);
    const float r0 = x0 - bf16_lo_f32(h), r1 = x1 - bf16_hi_f32(h);
    const uint32_t m = pack_bf16(r0, r1);
    ph[i] = h;
    pm[i] = m;
    pl[i] = pack_bf16(r0 - bf16_lo_f32(m), r1 - bf16_hi_f32(m));
  }
}

template <int AXIS, int K>
__global__ __launch_bounds__(512) void gram_pair16_kernel(const GramArgs a) {
  static_assert(K == 128 || K == 256, "quadrants of 128");
  constexpr int QUADS = K / 128;
  extern __shared__ __align__(16) unsigned char gsm[];
  const int b = blockIdx.x, qI = blockIdx.y / QUADS, qJ = blockIdx.y % QUADS;
  const int z = blockIdx.z;                      // (row-block within head, chunk)
  const int qi = z / a.nchunk, ch = z % a.nchunk;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 31, h = lane >> 5;
  const int64_t t0 = int64_t(ch) * a.chunk;
  const int64_t t1 = t0 + a.chunk < a.tlen ? t0 + a.chunk : a.tlen;
  const int64_t f0 = AXIS == CAFEQ_AXIS_COL ? int64_t(b) * K : (int64_t(b) * a.rep + qi) * K;
  const int64_t C = a.cols;

  // loader role: side (uniform over a wave), free index, half of the step's 16 contraction indices
  // (sixteen neighbouring lanes share a half and take consecutive free indices: their 16-byte LDS stores form one
  // contiguous 256-byte run, like the operand reads)
  // Along columns a wave takes 64 consecutive columns of one half; along rows it takes both halves of 32 rows, so
  // that the two 32-byte pieces of a row's 64 bytes are asked for by one instruction.
  const int side = __builtin_amdgcn_readfirstlane(tid >> 8);
  const int idx = AXIS == CAFEQ_AXIS_COL ? (tid & 127) : ((tid >> 6) & 3) * 32 + ((lane >> 5) << 4) + (lane & 15);
  const int half = AXIS == CAFEQ_AXIS_COL ? ((tid >> 7) & 1) : ((lane >> 4) & 1);
  const int64_t fbase = f0 + 128 * (side ? qJ : qI);     // uniform over the wave
  const int64_t fidx = fbase + idx;
  struct LoadSet {
    float lx[8], lsc[8];
    uint32_t lc[AXIS == CAFEQ_AXIS_COL ? 8 : 2];
    bool lok[AXIS == CAFEQ_AXIS_COL ? 8 : 2];
  };
  auto issue = [&](LoadSet& L, int64_t t) {
    const int64_t tt = t + 8 * half;
    if (AXIS == CAFEQ_AXIS_COL) {
      // uniform bases of the step's first row plus 32-bit lane offsets (rows past the chunk: its last row, dropped)
      const int64_t tb = t < t1 ? t : t1 - 1;            // (a step past the chunk: its last row, all dropped)
      const float* bx = a.X + tb * C + fbase;
      const int8_t* bc = a.codes + tb * C + fbase;
      const float* bs = a.scales + tb * (C / a.G);
      const int gcol = int(fidx / a.G), cg = int(C / a.G);
      const int rmax = t < t1 ? int(t1 - 1 - t < 15 ? t1 - 1 - t : 15) : -1;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r0 = 8 * half + e;
        L.lok[e] = r0 <= rmax;
        const int r = r0 <= rmax ? r0 : (rmax >= 0 ? rmax : 0);
        const uint32_t off = uint32_t(r) * uint32_t(C) + uint32_t(idx);
        L.lc[e] = uint32_t(uint8_t(bc[off]));
        L.lx[e] = bx[off];
        L.lsc[e] = bs[uint32_t(r) * uint32_t(cg) + uint32_t(gcol)];
      }
    } else {
      const int64_t grow = fidx / a.G;
#pragma unroll
      for (int q4 = 0; q4 < 2; ++q4) {
        const int64_t c = tt + 4 * q4;
        L.lok[q4] = c < t1;                               // tlen and chunk are multiples of 4
        const int64_t cc = L.lok[q4] ? c : t1 - 4;
        L.lc[q4] = *reinterpret_cast<const uint32_t*>(a.codes + fidx * C + cc);
        const float4 vx = *reinterpret_cast<const float4*>(a.X + fidx * C + cc);
        const float4 vs = *reinterpret_cast<const float4*>(a.scales + grow * C + cc);
        L.lx[4 * q4] = vx.x; L.lx[4 * q4 + 1] = vx.y; L.lx[4 * q4 + 2] = vx.z; L.lx[4 * q4 + 3] = vx.w;
        L.lsc[4 * q4] = vs.x; L.lsc[4 * q4 + 1] = vs.y; L.lsc[4 * q4 + 2] = vs.z; L.lsc[4 * q4 + 3] = vs.w;
      }
    }
  };
  auto commit = [&](const LoadSet& L, unsigned char* buf) {
    float q[8], er[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      bool ok;
      int code;
      if (AXIS == CAFEQ_AXIS_COL) { ok = L.lok[e]; code = int(int8_t(L.lc[e])); }
      else { ok = L.lok[e >> 2]; code = int(int8_t(L.lc[e >> 2] >> (8 * (e & 3)))); }
      const float v = __fmul_rn(float(code), L.lsc[e]);
      q[e] = ok ? v : 0.f;
      er[e] = ok ? v - L.lx[e] : 0.f;
    }
    uintx4 ph, pm, pl;
    split3_bf16(q, ph, pm, pl);
    unsigned char* dst = buf + (side ? 3 * kG16PlaneB : 0) + half * (kG16PlaneB / 2) + idx * 16;
    *reinterpret_cast<uintx4*>(dst) = ph;
    *reinterpret_cast<uintx4*>(dst + kG16PlaneB) = pm;
    *reinterpret_cast<uintx4*>(dst + 2 * kG16PlaneB) = pl;
    if (side) {
      split3_bf16(er, ph, pm, pl);
      *reinterpret_cast<uintx4*>(dst + 3 * kG16PlaneB) = ph;
      *reinterpret_cast<uintx4*>(dst + 4 * kG16PlaneB) = pm;
      *reinterpret_cast<uintx4*>(dst + 5 * kG16PlaneB) = pl;
    }
  };

  const int ta = wave >> 1, tc0 = 2 * (wave & 1);
  floatx16 accS[2], accR[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 16; ++v) { accS[u][v] = 0.f; accR[u][v] = 0.f; }

  auto products = [&](const unsigned char* buf) {
    const unsigned char* pa = buf + h * (kG16PlaneB / 2) + (ta * 32 + ln) * 16;
    bf16x8 ax[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) ax[p] = as_bf16x8(*reinterpret_cast<const uintx4*>(pa + p * kG16PlaneB));
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const unsigned char* pb = buf + 3 * kG16PlaneB + h * (kG16PlaneB / 2) + ((tc0 + u) * 32 + ln) * 16;
      bf16x8 bq[3], be[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        bq[p] = as_bf16x8(*reinterpret_cast<const uintx4*>(pb + p * kG16PlaneB));
        be[p] = as_bf16x8(*reinterpret_cast<const uintx4*>(pb + (3 + p) * kG16PlaneB));
      }
      // (smallest terms first)
      accS[u] = CAFEQ_MFMA_BF16(ax[1], bq[1], accS[u]);
      accS[u] = CAFEQ_MFMA_BF16(ax[0], bq[2], accS[u]);
      accS[u] = CAFEQ_MFMA_BF16(ax[2], bq[0], accS[u]);
      accS[u] = CAFEQ_MFMA_BF16(ax[0], bq[1], accS[u]);
      accS[u] = CAFEQ_MFMA_BF16(ax[1], bq[0], accS[u]);
      accS[u] = CAFEQ_MFMA_BF16(ax[0], bq[0], accS[u]);
      accR[u] = CAFEQ_MFMA_BF16(ax[1], be[1], accR[u]);
      accR[u] = CAFEQ_MFMA_BF16(ax[0], be[2], accR[u]);
      accR[u] = CAFEQ_MFMA_BF16(ax[2], be[0], accR[u]);
      accR[u] = CAFEQ_MFMA_BF16(ax[0], be[1], accR[u]);
      accR[u] = CAFEQ_MFMA_BF16(ax[1], be[0], accR[u]);
      accR[u] = CAFEQ_MFMA_BF16(ax[0], be[0], accR[u]);
    }
  };
  // Two steps of requests in flight (one register set per LDS buffer), and between two barriers a wave both
  // multiplies the step in one buffer and prepares the next step in the other (one barrier per step).  Requests
  // past the end of the chunk read in-range addresses and are dropped.
  LoadSet L0, L1;
  unsigned char* buf0 = gsm;
  unsigned char* buf1 = gsm + kG16BufB;
  issue(L0, t0);
  issue(L1, t0 + 16);
  commit(L0, buf0);
  for (int64_t t = t0; t < t1; t += 32) {
    __syncthreads();                       // buf0 holds step t; buf1's readers (step t - 16) are done
    issue(L0, t + 32);
    products(buf0);
    if (t + 16 < t1) {
      commit(L1, buf1);
      __syncthreads();                     // buf1 holds step t + 16; buf0's readers are done
      issue(L1, t + 48);
      products(buf1);
      if (t + 32 < t1) commit(L0, buf0);
    }
  }

  // partial[b][z][0|1][row][col]
  float* out = a.partial + ((size_t(b) * gridDim.z + z) * 2) * size_t(K) * K;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int col = 128 * qJ + (tc0 + u) * 32 + ln;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = 128 * qI + ta * 32 + 8 * (v / 4) + 4 * h + (v % 4);
      out[size_t(row) * K + col] = accS[u][v];
      out[size_t(K) * K + size_t(row) * K + col] = accR[u][v];
    }
  }
}

// The same pair for groups of 64 and more.  Along the contraction a value is code x scale, and a code is exact in ONE bfloat16 part, so
// with the scale s[t][group of i] taken over to the other operand,
//     S[i][j] = sum_t q[t][i] (s[t][i] Xq[t][j]),   R[i][j] = sum_t q[t][i] (s[t][i] E[t][j]),
// a product needs three part products instead of six, and the row side no split at all.  The right operands then belong to the row's
// group: V = 2 versions of them in a quadrant of 128 rows at groups of 64, one from 128 on.  Groups of 32 would need four versions, eight
// splits where the kernel above has three, and stay there.  The scales of i are multiplied by a power of two (and so are S and R, of
// which S^-1 R alone is used) that takes the square of the head's largest scale to about 1: the third parts of the right operands, products
// of two scales, then stay numbers in weights down to 2^-60, as far down as squares of float32 reach.  The largest of 64 scales stands
// for the head's: with 2^-64 to 2^64 as the factor's range no sum overflows that did not without it, unless all 64 are below a 2^-48th of it.
// (The head's first scale alone, without that range, turned a first line of 1e-37 next to ordinary ones into infinities.)
// A thread takes four contraction indices of one free index a step, for every version.  Along rows four lanes read a row's 64 bytes: 16
// cache lines a request.  With eight indices a thread (32 lines a request) the line lookups, 1024 and with the row side's codes 1280
// a step, were what the kernel took its time for: 104 us with six part products, 117 with three.
// 9B-shaped (V, O) pair, blocks of 256 and groups of 64: 62 + 104 -> 46.6 + 76.5 us.  Against float64 S is 8e-8 off (1.5e-7 with six
// products and their roundings), R 1.5e-7 (2.2e-7), S^-1 R 2.5e-7 (4e-7).
// Bound: a step's splits, LDS stores and matrix instructions between two barriers (2.9 k cycles along rows, of which matrix 0.8 k).
constexpr int kGqHalfB = 128 * 16 + 128;                       // a part's half of a step: 128 free indices x 8 bfloat16 (both halves' rows in other banks)
constexpr int kGqPlaneB = 2 * kGqHalfB;
constexpr size_t gq_buf(int V) { return size_t(1 + 6 * V) * kGqPlaneB; }   // the rows' codes; per version Xq and E in three parts
template <int AXIS, int K, int V>
__global__ __launch_bounds__(512) void gram_pair_codes_kernel(const GramArgs a) {
  static_assert((K == 128 || K == 256) && (V == 1 || V == 2), "quadrants of 128");
  constexpr int QUADS = K / 128;
  constexpr bool COL = AXIS == CAFEQ_AXIS_COL;
  extern __shared__ __align__(16) unsigned char gsm[];
  const int b = blockIdx.x, qI = blockIdx.y / QUADS, qJ = blockIdx.y % QUADS;
  const int z = blockIdx.z;                      // (row-block within head, chunk)
  const int qi = z / a.nchunk, ch = z % a.nchunk;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), ln = lane & 31, h = lane >> 5;
  const int64_t t0 = int64_t(ch) * a.chunk;
  const int64_t t1 = t0 + a.chunk < a.tlen ? t0 + a.chunk : a.tlen;
  const int64_t f0 = COL ? int64_t(b) * K : (int64_t(b) * a.rep + qi) * K;
  const int64_t C = a.cols, cg = C / a.G;
  float unit;                                    // 2^-2e, e the exponent of the largest of 64 of the head's scales (the same for all its workgroups)
  {
    const int64_t first = COL ? f0 : int64_t(b) * a.rep * K, g0 = first / a.G, g1 = (first + (COL ? K : a.rep * K) - 1) / a.G;
    const int64_t t = int64_t(lane) * a.tlen / 64, g = g0 + lane % (g1 - g0 + 1);
    const float m = cluster_allmax<64>(a.scales[COL ? t * cg + g : g * C + t]);
    const int e = int(__float_as_uint(m) >> 23 & 255) - 127;
    // (none of them but zeros: as if they were 2^-16, small enough for what cannot be seen and too large for nothing)
    unit = ldexpf(1.f, m > 0.f ? min(max(-2 * e, -64), 64) : 32);
  }

  // loader role: free index, quarter of the step's 16 contraction indices
  const int idx = COL ? (tid & 127) : tid >> 2, qt = COL ? (wave >> 1) : (tid & 3);
  const int64_t jbase = f0 + 128 * qJ, ibase = f0 + 128 * qI;
  // groups of this wave's columns (64 or 16 neighbours lie in one) and of the rows
  const int64_t gj = (jbase + (COL ? 64 * (wave & 1) : 16 * wave)) / a.G, gi0 = ibase / a.G, gi1 = V == 2 ? (ibase + 64) / a.G : gi0;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  int64_t gl = gj;                               // the group whose scales the lane asks for (columns)
  if ((lane >> 2 & 3) == 1) gl = gi0;
  if ((lane >> 2 & 3) > 1) gl = gi1;
  struct LoadSet {
    f32x4 lx, sj, si0, si1;                      // (columns: ls, a lane a scale, in place of sj and si)
    uintx4 lc, rc;                               // codes (rows: four in the first word)
    float ls;
    int ok;                                      // contraction indices of the thread's four that exist
  };
  auto issue = [&](LoadSet& L, int64_t t) __attribute__((always_inline)) {
    if (COL) {
      // uniform bases of the step's first row plus 32-bit lane offsets (rows past the chunk: its last row, dropped)
      const int64_t tb = t < t1 ? t : t1 - 1;
      const int rmax = t < t1 ? int(t1 - 1 - t < 15 ? t1 - 1 - t : 15) : -1, last = rmax >= 0 ? rmax : 0;
      const float* bx = a.X + tb * C + jbase;
      const int8_t *bc = a.codes + tb * C + jbase, *br = a.codes + tb * C + ibase;
      L.ok = rmax + 1 - 4 * qt;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * qt + e < last ? 4 * qt + e : last;
        const uint32_t off = uint32_t(r) * uint32_t(C) + uint32_t(idx);
        L.lc[e] = uint32_t(uint8_t(bc[off]));
        L.rc[e] = uint32_t(uint8_t(br[off]));
        L.lx[e] = bx[off];
      }
      // lanes 0 .. 3 the columns' scales of the quarter's rows, 4 .. 7 and 8 .. 11 the rows'
      const int r0 = 4 * qt + (lane & 3), r = r0 < last ? r0 : last;
      L.ls = a.scales[(tb + r) * cg + gl];
    } else {
      const int64_t tt = t + 4 * qt, c = tt < t1 ? tt : t1 - 4;       // tlen and chunk are multiples of 4
      L.ok = tt < t1 ? 4 : 0;
      L.lc[0] = *reinterpret_cast<const uint32_t*>(a.codes + (jbase + idx) * C + c);
      L.rc[0] = *reinterpret_cast<const uint32_t*>(a.codes + (ibase + idx) * C + c);
      L.lx = *reinterpret_cast<const f32x4*>(a.X + (jbase + idx) * C + c);
      L.sj = *reinterpret_cast<const f32x4*>(a.scales + gj * C + c);
      L.si0 = *reinterpret_cast<const f32x4*>(a.scales + gi0 * C + c);
      if (V == 2) L.si1 = *reinterpret_cast<const f32x4*>(a.scales + gi1 * C + c);
    }
  };
  // four values' three parts to one 8-byte place in each of three planes
  auto put = [](const float (&x)[4], unsigned char* at) __attribute__((always_inline)) {
    uint32_t p[3][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float x0 = x[2 * i], x1 = x[2 * i + 1];
      p[0][i] = pack_bf16(x0, x1);
      const float r0 = x0 - bf16_lo_f32(p[0][i]), r1 = x1 - bf16_hi_f32(p[0][i]);
      p[1][i] = pack_bf16(r0, r1);
      p[2][i] = pack_bf16(r0 - bf16_lo_f32(p[1][i]), r1 - bf16_hi_f32(p[1][i]));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(at + k * kGqPlaneB) = make_uint2(p[k][0], p[k][1]);
  };
  auto commit = [&](const LoadSet& L, unsigned char* buf) __attribute__((always_inline)) {
    unsigned char* dst = buf + (qt >> 1) * kGqHalfB + idx * 16 + (qt & 1) * 8;
    float xq[4], er[4], rcode[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int code = COL ? int(int8_t(L.lc[e])) : int(int8_t(L.lc[0] >> (8 * e)));
      const float sj = COL ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(L.ls), e)) : L.sj[e];
      xq[e] = __fmul_rn(float(code), sj);
      er[e] = xq[e] - L.lx[e];
      rcode[e] = float(COL ? int(int8_t(L.rc[e])) : int(int8_t(L.rc[0] >> (8 * e))));
      if (!(e < L.ok)) xq[e] = er[e] = 0.f;
    }
    *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16(rcode[0], rcode[1]), pack_bf16(rcode[2], rcode[3]));
#pragma unroll
    for (int v = 0; v < V; ++v) {
      float y[4], f[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float si = (COL ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(L.ls), 4 + 4 * v + e)) : v ? L.si1[e] : L.si0[e]) * unit;
        y[e] = xq[e] * si;
        f[e] = er[e] * si;
      }
      put(y, dst + (1 + 6 * v) * kGqPlaneB);
      put(f, dst + (4 + 6 * v) * kGqPlaneB);
    }
  };

  const int ta = wave >> 1, tc0 = 2 * (wave & 1);
  floatx16 accS[2], accR[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 16; ++v) { accS[u][v] = 0.f; accR[u][v] = 0.f; }
  auto products = [&](const unsigned char* buf) __attribute__((always_inline)) {
    const unsigned char* pa = buf + h * kGqHalfB + ln * 16;
    const bf16x8 ax = as_bf16x8(*reinterpret_cast<const uintx4*>(pa + ta * 512));
    bf16x8 bq[2][3], be[2][3];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const unsigned char* pb = pa + (1 + (V == 2 ? 6 * (ta >> 1) : 0)) * kGqPlaneB + (tc0 + u) * 512;
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        bq[u][p] = as_bf16x8(*reinterpret_cast<const uintx4*>(pb + p * kGqPlaneB));
        be[u][p] = as_bf16x8(*reinterpret_cast<const uintx4*>(pb + (3 + p) * kGqPlaneB));
      }
    }
    // (smallest terms first)
#pragma unroll
    for (int p = 2; p >= 0; --p)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        accS[u] = CAFEQ_MFMA_BF16(ax, bq[u][p], accS[u]);
        accR[u] = CAFEQ_MFMA_BF16(ax, be[u][p], accR[u]);
      }
  };
  // (buffers, requests and barriers as in the kernel above)
  LoadSet L0, L1;
  unsigned char* buf0 = gsm;
  unsigned char* buf1 = gsm + gq_buf(V);
  issue(L0, t0);
  issue(L1, t0 + 16);
  commit(L0, buf0);
  for (int64_t t = t0; t < t1; t += 32) {
    __syncthreads();                       // buf0 holds step t; buf1's readers (step t - 16) are done
    issue(L0, t + 32);
    products(buf0);
    if (t + 16 < t1) {
      commit(L1, buf1);
      __syncthreads();                     // buf1 holds step t + 16; buf0's readers are done
      issue(L1, t + 48);
      products(buf1);
      if (t + 32 < t1) commit(L0, buf0);
    }
  }

  // partial[b][z][0|1][row][col]
  float* out = a.partial + ((size_t(b) * gridDim.z + z) * 2) * size_t(K) * K;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int col = 128 * qJ + (tc0 + u) * 32 + ln;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = 128 * qI + ta * 32 + 8 * (v / 4) + 4 * h + (v % 4);
      out[size_t(row) * K + col] = accS[u][v];
      out[size_t(K) * K + size_t(row) * K + col] = accR[u][v];
    }
  }
}

// ---- paired quantization error from the Gram triples -------------------------------------------
// sums[(g)][m][K][K] (float64) = sum over the nchunk chunk partials of group g, m < 3
__global__ __launch_bounds__(256) void sum_triple_kernel(const float* __restrict__ partial, int nchunk, int K,
                                                          double* __restrict__ sums) {
  const int g = blockIdx.x, m = blockIdx.y;
  const size_t kk = size_t(K) * K;
  for (size_t e = size_t(blockIdx.z) * 256 + threadIdx.x; e < kk; e += size_t(gridDim.z) * 256) {
    double acc = 0.0;
    for (int c = 0; c < nchunk; ++c) acc += double(partial[((size_t(g) * nchunk + c) * 3 + m) * kk + e]);
    sums[(size_t(g) * 3 + m) * kk + e] = acc;
  }
}

// One workgroup per row-block q of V (head b = q / rep).  With SU = Uq^T Uq, RU = Uq^T E_U, TU = E_U^T E_U
// of head b and SV = Vq Vq^T, RV = Vq E_V^T, TV = E_V E_V^T of row-block q (E = dequantized - original):
//   Uq Vq - U V = Uq E_V + E_U V, so
//   ||Uq Vq - U V||_F^2 = tr(SU TV) + 2 tr(RU (RV - TV)) + tr(TU (SV - RV - RV^T + TV)),
//   ||U V||_F^2         = tr((SU - RU - RU^T + TU)(SV - RV - RV^T + TV));
// every term of the first line is at the scale of the rounding error (no cancellation).
__global__ __launch_bounds__(256) void pqe_trace_kernel(const double* __restrict__ su, const double* __restrict__ sv,
                                                         int K, int rep, double* __restrict__ perq) {
  __shared__ double red[2][4];
  const int q = blockIdx.x, b = q / rep;
  const size_t kk = size_t(K) * K;
  const double *SU = su + size_t(b) * 3 * kk, *RU = SU + kk, *TU = RU + kk;
  const double *SV = sv + size_t(q) * 3 * kk, *RV = SV + kk, *TV = RV + kk;
  double num = 0.0, den = 0.0;
  for (int e = threadIdx.x; e < K * K; e += 256) {
    const int i = e / K, j = e % K;
    const size_t ij = size_t(i) * K + j, ji = size_t(j) * K + i;
    const double vvt = SV[ji] - RV[ji] - RV[ij] + TV[ji];          // (V V^T)[j][i]
    const double utu = SU[ij] - RU[ij] - RU[ji] + TU[ij];          // (U^T U)[i][j]
    num += SU[ij] * TV[ji] + 2.0 * RU[ij] * (RV[ji] - TV[ji]) + TU[ij] * vvt;
    den += utu * vvt;
  }
  for (int m = 1; m < 64; m <<= 1) { num += __shfl_xor(num, m); den += __shfl_xor(den, m); }
  if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = num; red[1][threadIdx.x >> 6] = den; }
  __syncthreads();
  if (threadIdx.x == 0) {
    perq[2 * q] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    perq[2 * q + 1] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

__global__ void pqe_finish_kernel(const double* __restrict__ perq, int nq, float* __restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double num = 0.0, den = 0.0;
  for (int q = 0; q < nq; ++q) { num += perq[2 * q]; den += perq[2 * q + 1]; }
  out[0] = float(num);
  out[1] = float(den);
}

// The same inversion for a symmetric positive definite block of 256 in float32 (the Gram matrices of the adaptive
// rounding: diagonal pivots in natural order, so no permutation), as a block elimination in panels of 16 columns
// with everything but the 16 x 16 pivot block on the 16-bit matrix pipe.  With P the pivot block of panel t (rows
// and columns 16 t .. 16 t + 15 of the current matrix), D = P^-1, A the panel's other rows and X the sixteen pivot
// rows before the panel, sixteen elimination steps amount to
//     pivot block <- D,   panel (other rows) <- C = -A D,   pivot rows <- D X,   elsewhere  R <- R + C X,
// that is R += C' X on every row with C' = C (other rows) and D - I (pivot rows), and panel columns = C' + I.
// Only D needs the serial chain of steps (wave 0, one row per lane, pivot row through scalar lane reads; 16 lanes
// busy); C and the update are products of operands split exactly into three bfloat16 parts, the six part products
// of weight >= 2^-24 kept (as in gram_pair16_kernel).  Wave w of eight keeps rows 32 w .. 32 w + 31 as eight
// accumulator tiles: lane (ln, h) holds column 32 j + ln of tile j and rows 32 w + 8 (r / 4) + 4 h + r % 4,
// r = 0..15.  While wave 0 inverts P, the wave that holds the pivot rows (wave t / 2) splits them into the B
// operands of the update.  The contraction index c of the update is spread over the two lane halves as the
// accumulator layout delivers it -- half h takes c = 4 h + i and 8 + 4 h + i, i = 0..3 -- so that C^T = (-D^T) A^T
// comes out of the matrix pipe already in A-operand form (row 32 w + ln in lane ln), and the pivot rows' eight
// values per lane and tile are one 16-byte B operand; C in accumulator form, for the panel's own columns, is the
// same product with the operands exchanged.
__global__ __launch_bounds__(512) void gj_spd256_kernel(const GjArgs a) {
  constexpr int K = 256, NB = 16;
  __shared__ __align__(16) float pan[2][K][NB];
  constexpr int kXbB = 3 * 2 * K * 16;   // B operands of one panel's pivot rows: [part][lane half][column][8 rows]
  __shared__ __align__(16) unsigned char xb[2 * kXbB];
  __shared__ float dsm[2][16][17];       // D, float32
  __shared__ int deadflag, ready;        // ready: panels handed over so far
  __shared__ float wred[8];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, ln = lane & 31, h = lane >> 5;
  const int rbase = 32 * w + 4 * h;       // row of register r: rbase + 8 (r / 4) + r % 4
  floatx16 reg[8];
  if (a.partial == nullptr || a.sum32) {
    // (float32 input: all 128 requests of a lane land in their registers, none waits for a conversion)
    const float* src = (a.partial == nullptr ? a.T : a.sum32) + size_t(b) * K * K;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) reg[j][r] = src[(rbase + 8 * (r >> 2) + (r & 3)) * K + 32 * j + ln];
  } else if (a.sum64) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        reg[j][r] = float(a.sum64[size_t(b) * K * K + size_t(rbase + 8 * (r >> 2) + (r & 3)) * K + 32 * j + ln]);
  } else {
    const float* src = a.partial + size_t(b) * a.nz * 2 * K * K;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        double acc = 0;
        for (int z = 0; z < a.nz; ++z)
          acc += double(src[size_t(z) * 2 * K * K + size_t(rbase + 8 * (r >> 2) + (r & 3)) * K + 32 * j + ln]);
        reg[j][r] = float(acc);
      }
  }
  float anorm = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) anorm = fmaxf(anorm, fabsf(reg[j][r]));
  for (int m = 1; m < 64; m <<= 1) anorm = fmaxf(anorm, __shfl_xor(anorm, m));
  if (lane == 0) wred[w] = anorm;
  if (tid == 0) deadflag = 0;
  __syncthreads();
  anorm = 0;
  for (int i = 0; i < 8; ++i) anorm = fmaxf(anorm, wred[i]);
  int ex = 0;
  (void)frexp(double(anorm), &ex);
  const float scale = float(ldexp(1.0, -ex));    // exact power of two; 1 if the block is all zero
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) reg[j][r] *= scale;
  const float tol = anorm * scale * (a.partial ? 1e-5f : 1e-6f);

  // Two panels, one tile of columns, are a turn of the loop; between turns the tiles move down by one, so that register
  // indices are constants: reg[p] is tile (jt + p) % 8 in turn jt.  (All sixteen panels written out were 156 KB of code that ran
  // once and came from memory as it ran: 70.3 us, now 66.5.)
  // the panel's columns, as they are now, into pan[half] (lanes that hold them: ln - 16 half in 0..15)
  auto own_write = [&](auto half_c, auto p_c) __attribute__((always_inline)) {
    constexpr int half = decltype(half_c)::value, jt = decltype(p_c)::value;
    const int q_own = ln - NB * half;
    if (q_own >= 0 && q_own < NB) {
#pragma unroll
      for (int r = 0; r < 16; ++r) pan[half][rbase + 8 * (r >> 2) + (r & 3)][q_own] = reg[jt][r];
    }
  };
  // wave 0: D = P^-1, P = rows 16 t .. of pan[buf]; lane 16 g + r holds row r, columns 4 g .. of the pivot block, and, for the
  // four steps whose pivots they are, columns 4 q .. of its row too (sp), so that a step needs no other lanes than the sixteen
  // of its row: the pivot row's values come by DPP, eight multiply-adds a step.  (A whole row per lane, the pivot row through
  // scalar lane reads: sixteen of those and sixteen multiply-adds: solves of 75.3 instead of 70.3 us.)
  auto chain = [&](const int t, const int buf) __attribute__((always_inline)) {
    const int r = lane & 15, g = lane >> 4;
    float own[4], sp[4];
    {
      const float4 v = *reinterpret_cast<const float4*>(&pan[buf][NB * t + r][4 * g]);
      own[0] = v.x; own[1] = v.y; own[2] = v.z; own[3] = v.w;
    }
    bool dd = false;
    auto step = [&](auto s_c) __attribute__((always_inline)) {
      constexpr int s = decltype(s_c)::value, q = s / 4, e = s % 4;
      if constexpr (e == 0) {
        if constexpr (q > 0) {
#pragma unroll
          for (int c = 0; c < 4; ++c) own[c] = g == q - 1 ? sp[c] : own[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) sp[c] = __shfl(own[c], 16 * q + r);
      }
      const float pv = dpp_mov<0x150 + s>(sp[e]);             // row_newbcast: lane s of each sixteen
      dd = dd || !(pv > tol);
      // reciprocal of the pivot: hardware estimate (2^-22) + one Newton step
      float ipiv = __builtin_amdgcn_rcpf(pv);
      ipiv = ipiv * (2.f - pv * ipiv);
      const bool isp = r == s;
      const float f = (isp ? 1.f - pv : -sp[e]) * ipiv;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        own[c] = fmaf(f, dpp_mov<0x150 + s>(own[c]), own[c]);  // (columns 4 q ..: replaced by sp after their steps)
        sp[c] = c == e ? (isp ? 1.f : 0.f) + f : fmaf(f, dpp_mov<0x150 + s>(sp[c]), sp[c]);
      }
    };
    StaticFor<0, NB>::run(step);
#pragma unroll
    for (int c = 0; c < 4; ++c) dsm[buf][r][4 * g + c] = g == 3 ? sp[c] : own[c];
    if (dd && lane == 0) deadflag = 1;
  };
  // The wave that holds them splits the pivot rows 16 t + c, as they are now, into the B operands xb[half].
  // Lane (ln, h) holds, for each of its columns, c = 8 g + 4 h + i (g = 0, 1; i = 0..3) in register
  // 4 (2 half + g) + i: the eight contraction indices of lane half h, in operand order.
  auto publish = [&](auto half_c, const int jt) __attribute__((always_inline)) {
    constexpr int half = decltype(half_c)::value;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float xv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[e] = reg[j][8 * half + e];
      uintx4 xh, xm, xl;
      split3_bf16(xv, xh, xm, xl);
      unsigned char* dst = xb + half * kXbB + (h * K + 32 * ((jt + j) & 7) + ln) * 16;
      *reinterpret_cast<uintx4*>(dst) = xh;
      *reinterpret_cast<uintx4*>(dst + 2 * K * 16) = xm;
      *reinterpret_cast<uintx4*>(dst + 4 * K * 16) = xl;
    }
  };
  // Panel t = 2 jt + half, entered with pan[half], xb[half] and dsm[half] ready.  Every wave first updates the
  // tile that holds the next panel and hands that panel's columns over, so that wave 0 can invert the next pivot
  // block, after its own share of the update, while the slower waves are still multiplying: one barrier per panel.
  // (Measured without effect: a raised priority for wave 0; the inversion ahead of the rest of wave 0's update.)
  auto panel = [&](auto half_c, const int jt) __attribute__((always_inline)) {
    constexpr int half = decltype(half_c)::value, buf = half, nhalf = 1 - half, c0 = NB * half;
    constexpr int np = half;                 // the register tile of the next panel
    const int t = 2 * jt + half, nt = t + 1, njt = nt / 2;
    const bool has_next = nt < K / NB;
    const int q_own = ln - c0;
    const bool owner = q_own >= 0 && q_own < NB;
    float av[8], dv[8];
    const float4 a_lo = *reinterpret_cast<const float4*>(&pan[buf][32 * w + ln][8 * h]);
    const float4 a_hi = *reinterpret_cast<const float4*>(&pan[buf][32 * w + ln][8 * h + 4]);
    av[0] = a_lo.x; av[1] = a_lo.y; av[2] = a_lo.z; av[3] = a_lo.w;
    av[4] = a_hi.x; av[5] = a_hi.y; av[6] = a_hi.z; av[7] = a_hi.w;
#pragma unroll
    for (int e = 0; e < 8; ++e) dv[e] = owner ? -dsm[buf][8 * h + e][owner ? q_own : 0] : 0.f;
    uintx4 uh, um, ul;
    split3_bf16(av, uh, um, ul);
    const bf16x8 p0 = as_bf16x8(uh), p1 = as_bf16x8(um), p2 = as_bf16x8(ul);
    split3_bf16(dv, uh, um, ul);
    const bf16x8 d0 = as_bf16x8(uh), d1 = as_bf16x8(um), d2 = as_bf16x8(ul);
    floatx16 ct, cn;
#pragma unroll
    for (int v = 0; v < 16; ++v) { ct[v] = 0.f; cn[v] = 0.f; }
    // C^T (rows of the panel's columns c0 + c, column = this wave's row ln): operand order (-D^T, A^T)
    ct = CAFEQ_MFMA_BF16(d1, p1, ct);
    ct = CAFEQ_MFMA_BF16(d0, p2, ct);
    ct = CAFEQ_MFMA_BF16(d2, p0, ct);
    ct = CAFEQ_MFMA_BF16(d0, p1, ct);
    ct = CAFEQ_MFMA_BF16(d1, p0, ct);
    ct = CAFEQ_MFMA_BF16(d0, p0, ct);
    // C in accumulator form, valid in the owner lanes: operand order (A, -D)
    cn = CAFEQ_MFMA_BF16(p1, d1, cn);
    cn = CAFEQ_MFMA_BF16(p0, d2, cn);
    cn = CAFEQ_MFMA_BF16(p2, d0, cn);
    cn = CAFEQ_MFMA_BF16(p0, d1, cn);
    cn = CAFEQ_MFMA_BF16(p1, d0, cn);
    cn = CAFEQ_MFMA_BF16(p0, d0, cn);
    float cv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) cv[e] = ct[8 * half + e];
    if (w == jt && owner) {
      // this lane's row is pivot row q_own: D - I there
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int c = 8 * (e >> 2) + 4 * h + (e & 3);
        cv[e] = dsm[buf][q_own][c] - (c == q_own ? 1.f : 0.f);
      }
    }
    split3_bf16(cv, uh, um, ul);
    const bf16x8 a0 = as_bf16x8(uh), a1 = as_bf16x8(um), a2 = as_bf16x8(ul);
    auto update = [&](auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value;
      const unsigned char* pb = xb + buf * kXbB + (h * K + 32 * ((jt + j) & 7) + ln) * 16;
      const bf16x8 b0 = as_bf16x8(*reinterpret_cast<const uintx4*>(pb));
      const bf16x8 b1 = as_bf16x8(*reinterpret_cast<const uintx4*>(pb + 2 * K * 16));
      const bf16x8 b2 = as_bf16x8(*reinterpret_cast<const uintx4*>(pb + 4 * K * 16));
      // (smallest terms first)
      floatx16 d = reg[j];
      d = CAFEQ_MFMA_BF16(a1, b1, d);
      d = CAFEQ_MFMA_BF16(a0, b2, d);
      d = CAFEQ_MFMA_BF16(a2, b0, d);
      d = CAFEQ_MFMA_BF16(a0, b1, d);
      d = CAFEQ_MFMA_BF16(a1, b0, d);
      d = CAFEQ_MFMA_BF16(a0, b0, d);
      reg[j] = d;
    };
    auto others = [&](auto j_c) __attribute__((always_inline)) {
      if constexpr (decltype(j_c)::value != np) update(j_c);
    };
    update(std::integral_constant<int, np>{});
    if (has_next) {
      // (the next panel's columns lie in the other half of the lanes of this tile, or in the next one: the replacement of this
      // panel's own columns below does not touch them)
      own_write(std::integral_constant<int, nhalf>{}, std::integral_constant<int, np>{});
      // (every lane of the wave stores the count: each lane's own panel entries are released by its own store)
      if (w == njt) __hip_atomic_store(&ready, nt, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    StaticFor<0, 8>::run(others);
    // a panel column becomes the panel's own result: C' + I (D in the pivot rows)
    if (owner) {
#pragma unroll
      for (int r = 0; r < 16; ++r) cn[r] += (rbase + 8 * (r >> 2) + (r & 3)) == NB * t + q_own ? 1.f : 0.f;
      if (w == jt) {
#pragma unroll
        for (int e = 0; e < 8; ++e) cn[8 * half + e] = dsm[buf][8 * (e >> 2) + 4 * h + (e & 3)][q_own];
      }
      reg[0] = cn;
    }
    if (has_next) {
      if (w == njt) publish(std::integral_constant<int, nhalf>{}, jt);
      if (w == 0) {
        // the pivot block of the next panel is part of what wave njt handed over; the wait is bounded (a wave
        // that never saw the hand-over marks the block as failed and goes on)
        int spins = 0;
        while (__hip_atomic_load(&ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < nt && spins < (1 << 22)) {
          __builtin_amdgcn_s_sleep(1);
          ++spins;
        }
        if (spins >= (1 << 22) && lane == 0) deadflag = 1;
        chain(nt, nhalf);
      }
    }
    __syncthreads();
  };
  const std::integral_constant<int, 0> first{};
  const std::integral_constant<int, 1> second{};
  own_write(first, first);
  if (tid == 0) ready = 0;
  __syncthreads();
  if (w == 0) {
    chain(0, 0);
    publish(first, 0);
  }
  __syncthreads();
#pragma unroll 1
  for (int jt = 0; jt < K / 32; ++jt) {
    panel(first, jt);
    panel(second, jt);
    const floatx16 r0 = reg[0];
#pragma unroll
    for (int j = 0; j < 7; ++j) reg[j] = reg[j + 1];
    reg[7] = r0;
  }
  __syncthreads();
  const bool dead = deadflag != 0;
  if (a.status && tid == 0) a.status[size_t(b) * a.status_stride + a.status_offset] = dead ? 1 : 0;
  float* O = a.out + size_t(b) * K * K;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = rbase + 8 * (r >> 2) + (r & 3);
#pragma unroll
    for (int j = 0; j < 8; ++j) O[size_t(row) * K + 32 * j + ln] = dead ? 0.f : reg[j][r] * scale;
  }
}

// R_b = float64 sum over the chunk partials of the second matrix of each partial; C_b = I.
__global__ __launch_bounds__(256) void sum_r_init_c_kernel(const float* __restrict__ partial, int nz, int K,
                                                            float* __restrict__ R, float* __restrict__ C) {
  const int b = blockIdx.x;
  for (int e = blockIdx.y * 256 + threadIdx.x; e < K * K; e += gridDim.y * 256) {
    const float* p = partial + size_t(b) * nz * 2 * K * K + size_t(K) * K + e;
    double acc = 0;
    for (int z = 0; z < nz; ++z) acc += double(p[size_t(z) * 2 * K * K]);
    R[size_t(b) * K * K + e] = float(acc);
    C[size_t(b) * K * K + e] = (e / K == e % K) ? 1.f : 0.f;
  }
}


// Float64-accumulating batched product for the iterative refinement of the K = 256 solve:
// C_b (double) = alpha * A_b B_b + beta * C_b, A and B float or double, on the float64 matrix instruction
// (v_mfma_f64_16x16x4_f64: the vector pipe's float64 rate at a sixth of the operand traffic; a version on vector
// multiply-adds, 2 x 4 results per thread, was bound by its LDS reads: 18 us against 12-15).  A 32 x 64 tile per
// workgroup (the few blocks of a k = 256 workload then give one workgroup per compute unit) of four
// waves, wave w the 16 x 16 tiles (w / 2, 2 (w % 2)) and (w / 2, 2 (w % 2) + 1); chunks of 64 contraction indices
// through LDS, the next chunk's requests in flight while one is multiplied; K a multiple of 64.  (All four chunks
// of K = 256 requested at the start measured the same.)  Operand layouts: lane l gives A[i = l % 16][k = l / 16] and B[k = l / 16][j = l % 16];
// its four results are rows l / 16 + 4 r (r = 0..3) of column l % 16.
typedef double doublex4 __attribute__((ext_vector_type(4)));
// What becomes of the product: kF64Plain C = alpha A B + beta C; kF64Residual C = I - A B; kF64Step F = A + A B and
// kF64Solve F = I - (C + A B), rounded to float32 once (launches of their own for the identity, the sum and the difference
// took 5 us each).
// norms [block][tile] of the residual and the step: the tiles' shares of ||I - A B||_F^2.  kF64Residual writes them (null:
// it does not); kF64Step writes F2 as well as F where their sum is above kStepTwice2 (F2 null: never).  The Again variants,
// the second step of such blocks, leave every other block alone.
enum { kF64Plain, kF64Residual, kF64Step, kF64Solve, kF64ResidualAgain, kF64StepAgain };
constexpr float kStepTwice2 = 9e-8f;       // ||I - T X||_F <= 3e-4: its square is float32 rounding
constexpr int kF64Tiles256 = (256 / 32) * (256 / 64);
template <typename AT, typename BT, int EPI = kF64Plain>
__global__ __launch_bounds__(256) void bgemm_f64mfma_kernel(const AT* __restrict__ A, const BT* __restrict__ B,
                                                             double* __restrict__ C, int K, double alpha, double beta,
                                                             float* __restrict__ F, float* __restrict__ norms = nullptr,
                                                             float* __restrict__ F2 = nullptr) {
  constexpr bool RES = EPI == kF64Residual || EPI == kF64ResidualAgain, STEP = EPI == kF64Step || EPI == kF64StepAgain;
  constexpr int LC = 64;
  __shared__ double sa[32][LC + 2];   // [i][l]   (row strides chosen so that the operand reads of 32 lanes cover
  __shared__ double sb[LC][80];       // [l][j]    all banks once)
  const int tpc = K / 64, tpr = K / 32;
  int b, tile;
  block_and_part(blockIdx.x, tpr * tpc, gridDim.x, &b, &tile);
  const int i0 = (tile / tpc) * 32, j0 = (tile % tpc) * 64;
  bool twice = false;
  if constexpr (STEP || EPI == kF64ResidualAgain) {
    float t = 0.f;
#pragma unroll
    for (int q = 0; q < kF64Tiles256; ++q) t += norms[size_t(b) * kF64Tiles256 + q];
    twice = !(t <= kStepTwice2);               // uniform over the block
    if (EPI != kF64Step && !twice) return;
  }
  const AT* Ab = A + size_t(b) * K * K;
  const BT* Bb = B + size_t(b) * K * K;
  double* Cb = C + size_t(b) * K * K;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int ti = w >> 1, tj0 = 2 * (w & 1);
  doublex4 acc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[t][r] = 0.0;
  AT pa[8];
  BT pb[16];
  auto fetch = [&](int l0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = tid + 256 * q;
      pa[q] = Ab[(i0 + e / LC) * K + l0 + e % LC];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int e = tid + 256 * q;
      pb[q] = Bb[(l0 + e / 64) * K + j0 + e % 64];
    }
  };
  fetch(0);
  for (int l0 = 0; l0 < K; l0 += LC) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = tid + 256 * q;
      sa[e / LC][e % LC] = double(pa[q]);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int e = tid + 256 * q;
      sb[e / 64][e % 64] = double(pb[q]);
    }
    __syncthreads();
    if (l0 + LC < K) fetch(l0 + LC);
#pragma unroll
    for (int s4 = 0; s4 < LC / 4; ++s4) {
      const double av = sa[16 * ti + li][4 * s4 + lk];
      const double b0 = sb[4 * s4 + lk][16 * tj0 + li];
      const double b1 = sb[4 * s4 + lk][16 * (tj0 + 1) + li];
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b0, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b1, acc[1], 0, 0, 0);
    }
    __syncthreads();
  }
  float f2 = 0.f;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 16 * ti + lk + 4 * r, j = j0 + 16 * (tj0 + t) + li, at = i * K + j;
      if constexpr (EPI == kF64Plain) {
        Cb[at] = alpha * acc[t][r] + (beta != 0.0 ? beta * Cb[at] : 0.0);
      } else if constexpr (RES) {
        const double u = (i == j ? 1.0 : 0.0) - acc[t][r];
        Cb[at] = u;
        f2 = fmaf(float(u), float(u), f2);
      } else if constexpr (STEP) {
        const float u = float(double(Ab[at]) + acc[t][r]);
        F[size_t(b) * K * K + at] = u;
        if (EPI == kF64Step && twice && F2) F2[size_t(b) * K * K + at] = u;
      } else {
        F[size_t(b) * K * K + at] = float((i == j ? 1.0 : 0.0) - (acc[t][r] + Cb[at]));
      }
    }
  if constexpr (EPI == kF64Residual) {
    if (norms) {                               // (the LDS is free: a barrier ends the last chunk)
      float* red = reinterpret_cast<float*>(&sa[0][0]);
      f2 = wave_sum(f2);
      if (lane == 0) red[w] = f2;
      __syncthreads();
      if (tid == 0) norms[size_t(b) * kF64Tiles256 + tile] = (red[0] + red[1]) + (red[2] + red[3]);
    }
  }
}

// S64, R64 and a second copy of R64 (the residual's starting value) from the chunk partials; optionally S64
// rounded to float32.
// (eight partials of both matrices in flight per thread, one element each: with one at a time and eight elements a thread
// the 34 MB of the 9B-shaped (V, O) pair took 20 us, now 8)
__global__ __launch_bounds__(256) void sum_partials64_kernel(const float* __restrict__ partial, int nz, int K,
                                                              double* __restrict__ S64, double* __restrict__ R64,
                                                              double* __restrict__ res, float* __restrict__ S32) {
  const int b = blockIdx.x, e = blockIdx.y * 256 + threadIdx.x;   // (gridDim.y * 256 = K * K)
  const size_t kk = size_t(K) * K;
  const float* p = partial + size_t(b) * nz * 2 * kk + e;
  double s = 0, r = 0;
  int z = 0;
  for (; z + 8 <= nz; z += 8) {
    float u[8], v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) { u[q] = p[(z + q) * 2 * kk]; v[q] = p[((z + q) * 2 + 1) * kk]; }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 8; ++q) { s += double(u[q]); r += double(v[q]); }
  }
  for (; z < nz; ++z) { s += double(p[z * 2 * kk]); r += double(p[(z * 2 + 1) * kk]); }
  S64[b * kk + e] = s;
  if (S32) S32[b * kk + e] = float(s);
  R64[b * kk + e] = r;
  res[b * kk + e] = r;
}
// ---- blocks of 256 near a (scaled) rotation: Newton-Schulz rounds on the matrix cores before any elimination.
// X0 = T^T / alpha with alpha = ||T_b||_F^2 / K is the exact inverse of a rotation scaled by any factor and a
// good start near one.  grid (nb, K / 32): workgroup (b, s) writes rows 32 s .. of X0 (columns of T).
__global__ __launch_bounds__(1024) void ns_init_kernel(const float* __restrict__ T, float* __restrict__ X0, int K) {
  __shared__ float tile[256 * 33];
  __shared__ double red[16];
  const int b = blockIdx.x, s0 = blockIdx.y * 32, tid = threadIdx.x;
  const float* Tb = T + size_t(b) * K * K;
  double acc = 0;
  for (int e = tid * 4; e < K * K; e += 1024 * 4) {
    const float4 v = *reinterpret_cast<const float4*>(Tb + e);
    acc += double(v.x) * v.x + double(v.y) * v.y + double(v.z) * v.z + double(v.w) * v.w;
  }
  for (int m = 1; m < 64; m <<= 1) acc += __shfl_xor(acc, m);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  // tile[j][ii] = T[j][s0 + ii]
  for (int e = tid; e < K * 32; e += 1024) {
    const int j = e >> 5, ii = e & 31;
    tile[j * 33 + ii] = Tb[size_t(j) * K + s0 + ii];
  }
  __syncthreads();
  double f2 = 0;
  for (int w = 0; w < 16; ++w) f2 += red[w];
  const float inv_alpha = f2 > 0 ? float(double(K) / f2) : 0.f;
  float* Xb = X0 + size_t(b) * K * K;
  for (int e = tid; e < K * 32; e += 1024) {
    const int ii = e / K, j = e % K;
    Xb[size_t(s0 + ii) * K + j] = tile[j * 33 + ii] * inv_alpha;
  }
}
// One Newton round X' = X + X R, R = I - T X, of blocks of 256 in one launch: columns j of X' need columns j of R and all
// of X, columns j of R those of X and all of T, so a workgroup owns SL columns and streams T and X as matrix
// operands with no exchange between workgroups.  Eight waves, 32 rows each: a wave holds 16 rows of T (64 floats a lane)
// per tile, scales each row by a power of two and splits it into two float16 parts; the slice of X sits in LDS the
// same way (scaled per column), three part products (22 significant bits: R carries an error of about 1e-7 an entry).  The
// correction X R, second order in what its rounding loses, takes one part each.  What bounds it is the latency of 512 KB
// of operands per workgroup, and splitting them: 21 us for 8 blocks, 3-5 us when it copies.  (As two batched products on
// the float32 matrix pipe, with launches that measured the residual, a warm start took 12 launches and 107 us, now 7 and
// 75 us; 8 Adam steps on the 9B-shaped (V, O) pair 3700 -> 3085 us with the cold start's elimination avoided.)
// SL = 16 as long as those workgroups are at most one per compute unit (16 blocks), else 64, which split every row of T and
// X a quarter as often: a cold start 5 % off rotations takes 124 us for 8 blocks, 207 us for 32 and 674 us for 144 (149, 235
// and 842 us on the float32 products; sixteen columns for 144 blocks: nine rounds of workgroups a Newton round).
//   cur[b][256 / SL]: the slices' shares of ||R||_F^2.  prev: those of the round before (null: none).  A block whose last
//   measured residual was below 1e-3 (its correction left less than 1e-6 and the parts' 3e-5) or is beyond any contraction
//   to count on (||R||_F >= 3, a NaN) is copied, with its residual.  An entry that leaves float16's range makes R infinite.
constexpr float kNsAccept2 = 2.25e-4f;   // ||R||_F^2 before the last correction: 1.5e-2 leaves 2.3e-4 and what the parts lose
template <int SL>
struct NsRound {
  static constexpr int NC = SL / 16, NSL = 256 / SL, LD = 256 + 8;      // column tiles; slices per block; row of the LDS copies
  static constexpr size_t bytes = size_t(3) * SL * LD * 2 + (8 * SL + 8) * sizeof(float);
};
template <int SL>
__global__ __launch_bounds__(512) void ns256_round_kernel(const float* __restrict__ T, const float* __restrict__ X,
                                                          float* __restrict__ Xout, int nb, const float* __restrict__ prev,
                                                          float* __restrict__ cur) {
  constexpr int K = 256, LD = NsRound<SL>::LD, NC = NsRound<SL>::NC, NSL = NsRound<SL>::NSL;
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) unsigned char nsr_lds[];
  uint16_t* xh = reinterpret_cast<uint16_t*>(nsr_lds);   // X^T in two parts, R^T in one: [column][row]
  uint16_t* xl = xh + SL * LD;
  uint16_t* rh = xl + SL * LD;
  float* cmax = reinterpret_cast<float*>(rh + SL * LD);  // [8][SL]
  float* red = cmax + 8 * SL;
  const int b = int(blockIdx.x) % nb, sl = int(blockIdx.x) / nb, j0 = sl * SL;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 15, lg = lane >> 4;
  const float* Tb = T + size_t(b) * K * K;
  const float* Xb = X + size_t(b) * K * K;
  float* Ob = Xout + size_t(b) * K * K;
  // this thread's elements of the slice: columns 16 q + c .. + 7 of row l
  const int l = tid >> 1, c = (tid & 1) * 8;
  float4 sv[NC][2];
#pragma unroll
  for (int q = 0; q < NC; ++q)
#pragma unroll
    for (int u = 0; u < 2; ++u) sv[q][u] = *reinterpret_cast<const float4*>(Xb + l * K + j0 + 16 * q + c + 4 * u);
  if (prev) {
    float fp = 0.f;
    for (int q = 0; q < NSL; ++q) fp += prev[b * NSL + q];
    if (!(fp < 9.f) || fp <= 1e-6f) {            // uniform over the block
#pragma unroll
      for (int q = 0; q < NC; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u) *reinterpret_cast<float4*>(Ob + l * K + j0 + 16 * q + c + 4 * u) = sv[q][u];
      if (tid == 0) cur[b * NSL + sl] = sl == 0 ? fp : 0.f;
      return;
    }
  }
  // 16 rows of a matrix as A operands: lane (row ln, quarter lg) takes eight consecutive floats of every 32
  auto load_rows = [&](const float* M, int i, float4 (&u)[16]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float* p = M + (i + ln) * K + 32 * s + 8 * lg;
      u[2 * s] = *reinterpret_cast<const float4*>(p);
      u[2 * s + 1] = *reinterpret_cast<const float4*>(p + 4);
    }
  };
  // the power of two that puts a row's largest magnitude into [2^6, 2^7), and its inverse
  auto pow2_scale = [&](float m, float* inv) __attribute__((always_inline)) {
    int ex = int(__float_as_uint(m) >> 23);
    ex = ex < 40 ? 40 : (ex > 220 ? 220 : ex);
    *inv = __uint_as_float(uint32_t(ex - 6) << 23);
    return __uint_as_float(uint32_t(254 + 6 - ex) << 23);
  };
  auto row_scale = [&](const float4 (&u)[16], float* inv) __attribute__((always_inline)) {
    float m = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) m = fmaxf(fmaxf(m, fmaxf(fabsf(u[q].x), fabsf(u[q].y))), fmaxf(fabsf(u[q].z), fabsf(u[q].w)));
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    return pow2_scale(m, inv);
  };
  const int i0 = 32 * wave;
  float4 t0[16], t1[16];
  load_rows(Tb, i0, t0);
  load_rows(Tb, i0 + 16, t1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const float x[8] = {sv[q][0].x, sv[q][0].y, sv[q][0].z, sv[q][0].w, sv[q][1].x, sv[q][1].y, sv[q][1].z, sv[q][1].w};
    float m[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      m[e] = fabsf(x[e]);
#pragma unroll
      for (int o = 2; o < 64; o *= 2) m[e] = fmaxf(m[e], __shfl_xor(m[e], o));
    }
    if (lane < 2)
#pragma unroll
      for (int e = 0; e < 8; ++e) cmax[wave * SL + 16 * q + c + e] = m[e];
  }
  __syncthreads();
  auto column_max = [&](int j) __attribute__((always_inline)) {
    float m = cmax[j];
#pragma unroll
    for (int w = 1; w < 8; ++w) m = fmaxf(m, cmax[w * SL + j]);
    return m;
  };
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const float x[8] = {sv[q][0].x, sv[q][0].y, sv[q][0].z, sv[q][0].w, sv[q][1].x, sv[q][1].y, sv[q][1].z, sv[q][1].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int j = 16 * q + c + e;
      float inv;
      const float y = x[e] * pow2_scale(column_max(j), &inv);
      const _Float16 hi = _Float16(y), lo = _Float16(y - float(hi));
      xh[j * LD + l] = __builtin_bit_cast(uint16_t, hi);
      xl[j * LD + l] = __builtin_bit_cast(uint16_t, lo);
    }
  }
  float inv_c[NC];                               // this lane's columns
#pragma unroll
  for (int n = 0; n < NC; ++n) (void)pow2_scale(column_max(16 * n + ln), &inv_c[n]);
  __syncthreads();
  float f2 = 0.f;
  auto residual = [&](const float4 (&u)[16], int i) __attribute__((always_inline)) {
    float inv_r;
    const float sc = row_scale(u, &inv_r);
    floatx4 acc[NC], low[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) acc[n] = low[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float y[8] = {u[2 * s].x * sc, u[2 * s].y * sc, u[2 * s].z * sc, u[2 * s].w * sc,
                          u[2 * s + 1].x * sc, u[2 * s + 1].y * sc, u[2 * s + 1].z * sc, u[2 * s + 1].w * sc};
      halfx8 ah, al;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        ah[e] = _Float16(y[e]);
        al[e] = _Float16(y[e] - float(ah[e]));
      }
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        const halfx8 bh = as_halfx8(*reinterpret_cast<const uintx4*>(xh + (16 * n + ln) * LD + 32 * s + 8 * lg));
        const halfx8 bl = as_halfx8(*reinterpret_cast<const uintx4*>(xl + (16 * n + ln) * LD + 32 * s + 8 * lg));
        low[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, bh, low[n], 0, 0, 0);
        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bh, acc[n], 0, 0, 0);
        low[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bl, low[n], 0, 0, 0);
      }
    }
    float back[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) back[r] = __shfl(inv_r, 4 * lg + r);
    // element r: row i + 4 lg + r, column j0 + 16 n + ln
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      uint32_t p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float rv = (i + 4 * lg + r == j0 + 16 * n + ln ? 1.f : 0.f) - (acc[n][r] + low[n][r]) * (back[r] * inv_c[n]);
        f2 = fmaf(rv, rv, f2);
        p[r] = __builtin_bit_cast(uint16_t, _Float16(rv * 0x1p14f));
      }
      *reinterpret_cast<uint2*>(rh + (16 * n + ln) * LD + i + 4 * lg) = make_uint2(p[0] | (p[1] << 16), p[2] | (p[3] << 16));
    }
  };
  // (the rows of X for the correction are requested as soon as the rows of T have left their registers)
  residual(t0, i0);
  __builtin_amdgcn_sched_barrier(0);
  load_rows(Xb, i0, t0);
  __builtin_amdgcn_sched_barrier(0);
  residual(t1, i0 + 16);
  __builtin_amdgcn_sched_barrier(0);
  load_rows(Xb, i0 + 16, t1);
  float old[2][NC][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int n = 0; n < NC; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) old[t][n][r] = Xb[(i0 + 16 * t + 4 * lg + r) * K + j0 + 16 * n + ln];
  __builtin_amdgcn_sched_barrier(0);
  f2 = wave_sum(f2);
  if (lane == 0) red[wave] = f2;
  __syncthreads();
  if (tid == 0) {
    float t = red[0];
    for (int w = 1; w < 8; ++w) t += red[w];
    cur[b * NSL + sl] = t;
  }
  auto correct = [&](const float4 (&u)[16], int i, const float (&o)[NC][4]) __attribute__((always_inline)) {
    float inv_r;
    const float sc = row_scale(u, &inv_r);
    floatx4 acc[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) acc[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float y[8] = {u[2 * s].x * sc, u[2 * s].y * sc, u[2 * s].z * sc, u[2 * s].w * sc,
                          u[2 * s + 1].x * sc, u[2 * s + 1].y * sc, u[2 * s + 1].z * sc, u[2 * s + 1].w * sc};
      halfx8 ah;
#pragma unroll
      for (int e = 0; e < 8; ++e) ah[e] = _Float16(y[e]);
#pragma unroll
      for (int n = 0; n < NC; ++n)
        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
            ah, as_halfx8(*reinterpret_cast<const uintx4*>(rh + (16 * n + ln) * LD + 32 * s + 8 * lg)), acc[n], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float back = __shfl(inv_r, 4 * lg + r) * 0x1p-14f;
#pragma unroll
      for (int n = 0; n < NC; ++n) Ob[(i + 4 * lg + r) * K + j0 + 16 * n + ln] = fmaf(acc[n][r], back, o[n][r]);
    }
  };
  correct(t0, i0, old[0]);
  correct(t1, i0 + 16, old[1]);
}

}  // namespace

namespace {
int launch_gj(const GjArgs& a, int nb, hipStream_t st) {
  // the Gram matrices of the adaptive rounding are symmetric positive definite: no pivot search there; only the
  // blockwise inverse of blocks of 256 comes here with general ones (inverse_kernels.hip has the smaller blocks)
  switch (a.K) {
    case 32: hipLaunchKernelGGL((gj_panel_kernel<32, 4, 4, double, false>), dim3(nb), dim3(64), 0, st, a); break;
    case 64: hipLaunchKernelGGL((gj_panel_kernel<64, 4, 8, double, false>), dim3(nb), dim3(128), 0, st, a); break;
    case 128: hipLaunchKernelGGL((gj_panel_kernel<128, 4, 8, double, false>), dim3(nb), dim3(512), 0, st, a); break;
    case 256:
      if (a.partial == nullptr) hipLaunchKernelGGL((gj_panel_kernel<256, 8, 16, float, true>), dim3(nb), dim3(512), 0, st, a);
      else hipLaunchKernelGGL(gj_spd256_kernel, dim3(nb), dim3(512), 0, st, a);
      break;
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
}  // namespace

int launch_gram(int axis, const float* X, const int8_t* codes, const float* scales, int64_t rows, int64_t cols,
                int K, int G, int nb, int rep, int64_t chunk, int nchunk, bool triple, float* partial, hipStream_t st);
int launch_gram_pair(int axis, const float* X, const int8_t* codes, const float* scales, int64_t rows,
                     int64_t cols, int K, int G, int nb, int rep, int64_t chunk, int nchunk, float* partial,
                     hipStream_t st) {
  return launch_gram(axis, X, codes, scales, rows, cols, K, G, nb, rep, chunk, nchunk, false, partial, st);
}
// Paired quantization error from Gram triples.  partialU / partialV: 3 k x k matrices per (head, chunk) /
// (row-block, chunk); sums: 3 * (nb + nb*rep) * k * k doubles + 2 * nb * rep doubles.
int launch_pqe(const float* U, const float* V, int64_t rowsA, int64_t colsA, int64_t rowsB, int64_t colsB, int K,
               int GA, int GB, int nb, int rep, const int8_t* codesU, const float* scalesU, const int8_t* codesV,
               const float* scalesV, int64_t chunkA, int nchunkA, int64_t chunkB, int nchunkB, float* partialU,
               float* partialV, double* sums, float* out, hipStream_t st) {
  int rc = launch_gram(CAFEQ_AXIS_COL, U, codesU, scalesU, rowsA, colsA, K, GA, nb, 1, chunkA, nchunkA, true, partialU, st);
  if (rc) return rc;
  rc = launch_gram(CAFEQ_AXIS_ROW, V, codesV, scalesV, rowsB, colsB, K, GB, nb, rep, chunkB, nchunkB, true, partialV, st);
  if (rc) return rc;
  const size_t kk = size_t(K) * K;
  double* su = sums;
  double* sv = sums + size_t(nb) * 3 * kk;
  double* perq = sv + size_t(nb) * rep * 3 * kk;
  hipLaunchKernelGGL(sum_triple_kernel, dim3(nb, 3, 16), dim3(256), 0, st, partialU, nchunkA, K, su);
  hipLaunchKernelGGL(sum_triple_kernel, dim3(nb * rep, 3, 16), dim3(256), 0, st, partialV, nchunkB, K, sv);
  hipLaunchKernelGGL(pqe_trace_kernel, dim3(nb * rep), dim3(256), 0, st, su, sv, K, rep, perq);
  hipLaunchKernelGGL(pqe_finish_kernel, dim3(1), dim3(64), 0, st, perq, nb * rep, out);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
int launch_gram(int axis, const float* X, const int8_t* codes, const float* scales, int64_t rows, int64_t cols,
                int K, int G, int nb, int rep, int64_t chunk, int nchunk, bool triple, float* partial, hipStream_t st) {
  GramArgs a;
  a.X = X; a.codes = codes; a.scales = scales; a.rows = rows; a.cols = cols; a.K = K; a.G = G;
  a.rep = axis == CAFEQ_AXIS_COL ? 1 : rep;
  a.tlen = axis == CAFEQ_AXIS_COL ? rows : cols;
  a.chunk = chunk; a.nchunk = nchunk; a.partial = partial;
  if (!triple && (K == 128 || K == 256)) {
    // heads of 128 and 256: the 16-bit kernels, one workgroup per (head, quadrant of 128 x 128, chunk)
    const dim3 g16(nb, (K / 128) * (K / 128), a.rep * nchunk);
    static std::atomic<bool> attr_set{false};
    const size_t lds = G % 64 ? kG16Lds : 2 * gq_buf(G == 64 ? 2 : 1);
    bool ok = true;
    const bool set = !attr_set;
    auto run = [&](auto kern, bool mine) {
      if (set) ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 2 * int(gq_buf(2))) == hipSuccess;
      if (mine && ok) hipLaunchKernelGGL(kern, g16, dim3(512), lds, st, a);
    };
#define CAFEQ_GRAM16(AX, KK)                                                        \
  {                                                                                 \
    const bool here = axis == AX && K == KK;                                        \
    run(gram_pair16_kernel<AX, KK>, here && G % 64 != 0);                           \
    run(gram_pair_codes_kernel<AX, KK, 1>, here && G % 64 == 0 && G != 64);         \
    run(gram_pair_codes_kernel<AX, KK, 2>, here && G == 64);                        \
  }
    CAFEQ_GRAM16(CAFEQ_AXIS_COL, 128) CAFEQ_GRAM16(CAFEQ_AXIS_COL, 256)
    CAFEQ_GRAM16(CAFEQ_AXIS_ROW, 128) CAFEQ_GRAM16(CAFEQ_AXIS_ROW, 256)
#undef CAFEQ_GRAM16
    if (!ok) return CAFEQ_ERR_LAUNCH;
    attr_set = true;
    CAFEQ_CHECK_LAUNCH();
    return CAFEQ_OK;
  }
  dim3 grid(nb, K / 32, a.rep * nchunk);
#define CAFEQ_GRAM(KK)                                                                                          \
  case KK:                                                                                                      \
    if (axis == CAFEQ_AXIS_COL) {                                                                               \
      if (triple) hipLaunchKernelGGL((gram_pair_kernel<CAFEQ_AXIS_COL, KK, true>), grid, dim3(256), 0, st, a);  \
      else hipLaunchKernelGGL((gram_pair_kernel<CAFEQ_AXIS_COL, KK, false>), grid, dim3(256), 0, st, a);        \
    } else {                                                                                                    \
      if (triple) hipLaunchKernelGGL((gram_pair_kernel<CAFEQ_AXIS_ROW, KK, true>), grid, dim3(256), 0, st, a);  \
      else hipLaunchKernelGGL((gram_pair_kernel<CAFEQ_AXIS_ROW, KK, false>), grid, dim3(256), 0, st, a);        \
    }                                                                                                           \
    break;
  switch (K) {
    CAFEQ_GRAM(32) CAFEQ_GRAM(64) CAFEQ_GRAM(128) CAFEQ_GRAM(256)
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
#undef CAFEQ_GRAM
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}

// C_b = I - S_b^-1 R_b with S, R the float64 sums of the chunk partials.  Sinv, R: [nb][K][K]
// float32 scratch; work: 4 * nb * K * K doubles.  A singular S_b yields C_b = I and status 1.
// K <= 128: S is inverted in float64.  K == 256: S is inverted in float32 and the solution
// X = S^-1 R gets one step of iterative refinement with float64 residuals.
int launch_gj_solve(int K, int nb, int nz, const float* partial, double* work, float* Sinv, float* R,
                    float* out, int* status, int status_stride, int status_offset, hipStream_t st) {
  GjArgs a;
  a.K = K; a.nz = nz; a.T = nullptr; a.partial = partial; a.out = Sinv;
  a.status = status; a.status_stride = status_stride;
  a.status_offset = status_offset;
  const size_t mat = size_t(nb) * K * K;
  double *S64 = work, *R64 = work + mat, *res = work + 2 * mat, *X64 = work + 3 * mat;
  if (K == 256 || nb <= 64) {
    // few blocks (always so for K = 256 shapes): the sums over the chunk partials are formed by the whole chip
    // (K == 256 does not use the float32 scratch R otherwise: it holds the rounded sum the elimination reads)
    float* S32 = K == 256 ? R : nullptr;
    hipLaunchKernelGGL(sum_partials64_kernel, dim3(nb, K * K / 256), dim3(256), 0, st, partial, nz, K, S64, R64, res, S32);
    CAFEQ_CHECK_LAUNCH();
    a.sum64 = S64;
    a.sum32 = S32;
  }
  int rc = launch_gj(a, nb, st);
  if (rc) return rc;
  if (K < 256) {
    hipLaunchKernelGGL(sum_r_init_c_kernel, dim3(nb, 16), dim3(256), 0, st, partial, nz, K, R, out);
    CAFEQ_CHECK_LAUNCH();
    return launch_bgemm(false, false, Sinv, R, out, K, nb, -1.f, 1.f, st);
  }
  const unsigned grid = unsigned(nb) * (K / 32) * (K / 64);
  hipLaunchKernelGGL((bgemm_f64mfma_kernel<float, double>), dim3(grid), dim3(256), 0, st, Sinv, R64, X64, K, 1.0, 0.0,
                     static_cast<float*>(nullptr));
  hipLaunchKernelGGL((bgemm_f64mfma_kernel<double, double>), dim3(grid), dim3(256), 0, st, S64, X64, res, K, -1.0, 1.0,
                     static_cast<float*>(nullptr));
  hipLaunchKernelGGL((bgemm_f64mfma_kernel<float, double, kF64Solve>), dim3(grid), dim3(256), 0, st, Sinv, res, X64, K, 1.0,
                     1.0, out);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}

// Blocks of 256.  Newton rounds (ns256_round_kernel) from X0 = T^T / alpha (cold: up to five) or from the inverse already
// in Tinv (warm: inside a learning loop, two), used per block when the residual measured before the last correction is at
// most 1.5e-2: a round squares it and adds what its 16-bit operands lose, 2^-12 of it times ||T|| ||X||, which shows in the
// residual before (its own parts lose 2^-23 of ||T|| ||X||) long before it could undo the contraction; a block that meets
// the bound early is copied through the rest.  Every other block is eliminated in float32 (one compute unit each, 283 us).
// Either way the float64 residual of the X at hand follows and a Newton step with it, which squares it; where that residual
// is above 3e-4 (conditions from several hundred on, whichever way X came about), a second one.  With one step alone
// eliminated blocks of condition 1e3 were 1.1e-6 off, of 1e4 1.2e-4; now 2.6e-8.  Blocks that need no second step pay
// two launches that return at once.
// Five rounds: they reach blocks with ||I - T X0||_2 up to about 0.7 (three left 0.05-perturbed rotations next to the
// elimination, whose 283 us one block of a call is enough to pay).
// work: 2 nb K K doubles: the float64 residual (before it the rounds' residual norms), then two float32 matrices; and
// nb kF64Tiles256 floats, the float64 residual's norms.
size_t inverse256_workspace_bytes(int nb) { return size_t(nb) * (size_t(2) * 256 * 256 * sizeof(double) + kF64Tiles256 * sizeof(float)); }
int launch_inverse256(const float* T, int nb, double* work, float* Tinv, float* rho_row, float* rho_col, int* status,
                      bool warm, hipStream_t st) {
  constexpr int K = 256, kCold = 5, kWarm = 2;
  int rc;
  const size_t mat = size_t(nb) * K * K;
  double* res = work;
  float* buf[2] = {reinterpret_cast<float*>(work + mat), reinterpret_cast<float*>(work + mat) + mat};
  float* norms = reinterpret_cast<float*>(work);             // [round][nb][slices]
  const bool narrow = int64_t(nb) * NsRound<16>::NSL <= device_cu_count();
  const int nsl = narrow ? NsRound<16>::NSL : NsRound<64>::NSL;
  static std::atomic<bool> attr_set{false};
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(ns256_round_kernel<64>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            int(NsRound<64>::bytes)) != hipSuccess)
      return CAFEQ_ERR_LAUNCH;
    attr_set = true;
  }
  if (!warm) hipLaunchKernelGGL(ns_init_kernel, dim3(nb, K / 32), dim3(1024), 0, st, T, buf[0], K);
  const int rounds = warm ? kWarm : kCold;
  const float* X = warm ? Tinv : buf[0];
  for (int r = 0; r < rounds; ++r) {
    float* Xn = X == buf[0] ? buf[1] : buf[0];
    const float* prev = r ? norms + size_t(r - 1) * nb * nsl : nullptr;
    float* cur = norms + size_t(r) * nb * nsl;
    if (narrow)
      hipLaunchKernelGGL(ns256_round_kernel<16>, dim3(unsigned(nb) * nsl), dim3(512), NsRound<16>::bytes, st, T, X, Xn, nb, prev, cur);
    else
      hipLaunchKernelGGL(ns256_round_kernel<64>, dim3(unsigned(nb) * nsl), dim3(512), NsRound<64>::bytes, st, T, X, Xn, nb, prev, cur);
    X = Xn;
  }
  CAFEQ_CHECK_LAUNCH();
  GjArgs a;
  a.K = K; a.nz = 0; a.T = T; a.partial = nullptr; a.out = const_cast<float*>(X);
  a.status = status; a.status_stride = 1; a.status_offset = 0;
  a.resid = norms + size_t(rounds - 1) * nb * nsl; a.nresid = nsl; a.resid_max = kNsAccept2;
  if ((rc = launch_gj(a, nb, st))) return rc;
  // Newton steps X <- X + X (I - T X) with float64 residuals
  const unsigned grid = unsigned(nb) * (K / 32) * (K / 64);
  float* rnorm = reinterpret_cast<float*>(work + 2 * mat);
  float* X1 = X == buf[0] ? buf[1] : buf[0];
  hipLaunchKernelGGL((bgemm_f64mfma_kernel<float, float, kF64Residual>), dim3(grid), dim3(256), 0, st, T, X, res, K, 1.0, 0.0,
                     static_cast<float*>(nullptr), rnorm);
  hipLaunchKernelGGL((bgemm_f64mfma_kernel<float, double, kF64Step>), dim3(grid), dim3(256), 0, st, X, res,
                     static_cast<double*>(nullptr), K, 1.0, 0.0, Tinv, rnorm, X1);
  hipLaunchKernelGGL((bgemm_f64mfma_kernel<float, float, kF64ResidualAgain>), dim3(grid), dim3(256), 0, st, T, X1, res, K, 1.0,
                     0.0, static_cast<float*>(nullptr), rnorm);
  hipLaunchKernelGGL((bgemm_f64mfma_kernel<float, double, kF64StepAgain>), dim3(grid), dim3(256), 0, st, X1, res,
                     static_cast<double*>(nullptr), K, 1.0, 0.0, Tinv, rnorm);
  CAFEQ_CHECK_LAUNCH();
  RhoRequest rho[2];
  int nrho = 0;
  if (rho_row) rho[nrho++] = RhoRequest{Tinv, rho_row, 1};
  if (rho_col) rho[nrho++] = RhoRequest{Tinv, rho_col, 0};
  if (nrho && (rc = launch_split_planes_multi(nullptr, 0, K, nb, st, nullptr, 0, rho, nrho))) return rc;
  return CAFEQ_OK;
}

}  // namespace cafeq
