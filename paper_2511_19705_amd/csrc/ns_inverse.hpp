// Newton's iteration for one transform block per workgroup: the body of the inverse's own kernels and, inside a learning loop over
// blocks of 32, of what follows the update (inverse_kernels.hip says why products, and what they measure).
#pragma once
#include "gj_panel.hpp"

namespace cafeq {

// what a float16 pair (pack_f16: rounded to nearest, a magnitude beyond float16's range to infinity) leaves of (x0, x1)
__device__ __forceinline__ uint32_t pack_f16_rest(float x0, float x1, uint32_t hi) {
  const halfx2 p = __builtin_bit_cast(halfx2, hi);
  return pack_f16(x0 - float(p[0]), x1 - float(p[1]));
}

// Four signed bytes d1..d4 of round(x 2^30), |x| < 1: x = d1 2^-6 + d2 2^-14 + d3 2^-22 + d4 2^-30 up to 2^-31 (exact
// down to 2^-7), as bytes 3..0 of a word.
__device__ __forceinline__ uint32_t digits_of(float x) {
  return (uint32_t(int(__builtin_rintf(x * 0x1p30f))) + 0x00808080u) ^ 0x00808080u;
}
// digits of four values -> one word per digit, the values' bytes in order
__device__ __forceinline__ void digit_words(const float (&x)[4], uint32_t (&d)[4]) {
  const uint32_t w0 = digits_of(x[0]), w1 = digits_of(x[1]), w2 = digits_of(x[2]), w3 = digits_of(x[3]);
  const uint32_t lo01 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), hi01 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
  const uint32_t lo23 = __builtin_amdgcn_perm(w3, w2, 0x05010400u), hi23 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
  d[3] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
  d[2] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
  d[1] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
  d[0] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
}
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx16 __attribute__((ext_vector_type(16)));

// Newton's iteration for one block per workgroup, a wave keeps its tiles of X in float32
// registers and its 32 rows of T as A operands.  R = I - T X runs on two float16 parts per operand, three products
// (22 significant bits: R carries an absolute error of about 1e-7, its Frobenius norm of 1e-5 at k = 128); the
// correction X R, second order in what its rounding loses, on one part each.  T and X are scaled by powers of two
// that keep the parts inside float16's range; an entry that leaves it has an infinite high and an opposite infinite low
// part, their column of R is not a number, and no bound accepts that.  (The parts are rounded to nearest.  Rounded towards
// zero they saturate, and R belongs to another X than the one that is updated.)
// LDS: X^T in two parts and R^T in one, as the accumulator layout delivers them (four consecutive rows of a column per
// lane), and X in one part: 136 KB at k = 128.
//   WARM 0: start from T^T / alpha.  WARM 1: start from the inverse already in Tinv.
// The round that starts at ||R||_F <= 3e-3 is the last; one Newton step with an exact residual follows, which measures
// ||R||_F <= 2e-5 (else the block is eliminated) and leaves its square: the result carries its rounding to float32 only,
// like the float64 elimination's.
// The exact residual runs on the 8-bit integer matrix pipe: T and X as four signed base-256 digits of 31-bit
// fixed-point values, the thirteen digit products of weight >= 2^-44 summed in 32-bit integers, one sum a weight, and the
// sums taken from the identity one after the other.  That is 1.7 k cycles per 32 x 32 tile
// at k = 128; v_mfma_f64_16x16x4_f64, which sustains about a third of its published rate here, took 25 k (29 us
// for 112 blocks even on four workgroups per block).
// A block of 64 or 128 that is a rotation to float32 accuracy (max |I - T T^T| <= 2e-6) gets T^T itself.
// tiles of 32 columns per wave: at k = 128 two, so that eight waves have the registers for their rows of T (sixteen
// waves of one tile spilled 35)
template <int K>
struct NsShape {
  static constexpr int TPW = K == 128 ? 2 : 1, NTL = K / 32, NWJ = NTL / TPW, NW = NTL * NWJ, LDH = K + 8;
  static constexpr int LDG = K + 16;     // bytes per row of a digit of X^T
  static constexpr size_t it = size_t(4) * K * LDH * 2 + 2 * NW * sizeof(float), gj = sizeof(GjShared<K, double>);
  static constexpr size_t bytes = it > gj ? it : gj;
  static_assert(4 * K * LDG <= 3 * K * LDH * 2, "the digits lie over X^T and R^T");
  static constexpr int LDS = K + 4;      // floats per row of T on its way to the registers
  // log2 max|T| max|X| up to which the exact residual's digits are used.  At k = 32, where the elimination costs no more than
  // two rounds, as far as they reach its precision (off float64 2.5e-8 in the root mean square; condition 10 is 1, at 100
  // 2.57e-8, at 1000 3.8e-8).  64 and 128 are bounded by the residual they measure, which eliminates from condition 300 or
  // so on (2.58e-8 at condition 100); 9: what float16 holds of X.
  static constexpr int kMaxShift = K == 32 ? 1 : 9;
  static_assert(K * LDS * 4 <= 3 * K * LDH * 2, "and so does T");
};
// ns_lds: NsShape<K>::bytes; threads NsShape<K>::NW * 64 of the workgroup, the others of it, if any, have ended.
// false: the block is to be eliminated, by the kernel itself, in the same LDS (ns_eliminate_args).  From in here gj_panel_body, a function of
// its own at k = 128, would get a pointer of which the compiler has lost that it is LDS: 8 blocks of 128 far from rotations 99 -> 132 us.
template <int K, int WARM>
__device__ __forceinline__ bool ns_inverse_body(const float* __restrict__ T, float* __restrict__ Tinv, int* __restrict__ status, const int b,
                                                unsigned char* ns_lds) {
  using S = NsShape<K>;
  constexpr int TPW = S::TPW, NW = S::NW, LDH = S::LDH, NS = K / 16, kMaxRounds = 10;
  uint16_t* xth = reinterpret_cast<uint16_t*>(ns_lds);   // X^T[j][i], high and low parts
  uint16_t* xtl = xth + K * LDH;
  uint16_t* rt = xtl + K * LDH;                           // R^T[j][i]
  uint16_t* xr = rt + K * LDH;                            // X[i][j], high part
  float* red = reinterpret_cast<float*>(xr + K * LDH);    // [2][NW]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ln = lane & 31, h = lane >> 5, i0 = 32 * (wave / S::NWJ) + 4 * h, j0 = 32 * TPW * (wave % S::NWJ) + ln;
  const float* Tb = T + size_t(b) * K * K;
  float* Ob = Tinv + size_t(b) * K * K;

  // T into LDS, whole rows at a time (a lane's own accesses, 16 bytes of 64 different rows per request, cost the start
  // of the kernel 20 k cycles)
  float* stage = reinterpret_cast<float*>(ns_lds);
  constexpr int kStage = K * K / 4 / (NW * 64);
  auto stage_t = [&]() __attribute__((always_inline)) {
    float4 u[kStage];
#pragma unroll
    for (int q = 0; q < kStage; ++q) u[q] = *reinterpret_cast<const float4*>(Tb + (tid + q * NW * 64) * 4);
#pragma unroll
    for (int q = 0; q < kStage; ++q) {
      const int e = (tid + q * NW * 64) * 4;
      *reinterpret_cast<float4*>(stage + (e / K) * S::LDS + e % K) = u[q];
    }
  };
  const float* trow = stage + (i0 - 4 * h + ln) * S::LDS;   // this lane's row of T as an A operand
  stage_t();
  __syncthreads();
  // this wave's tiles of T^T: element v of tile t is row i0 + 8 (v / 4) + v % 4, column j0 + 32 t
  float x[TPW][16];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 u = *reinterpret_cast<const float4*>(stage + (j0 + 32 * t) * S::LDS + i0 + 8 * g);
      x[t][4 * g] = u.x; x[t][4 * g + 1] = u.y; x[t][4 * g + 2] = u.z; x[t][4 * g + 3] = u.w;
    }
  float am = 0.f, f2 = 0.f;
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      am = fmaxf(am, fabsf(x[t][v]));
      f2 = fmaf(x[t][v], x[t][v], f2);
    }
  am = cluster_allmax<64>(am);
  f2 = wave_sum(f2);
  if (lane == 0) { red[wave] = am; red[NW + wave] = f2; }
  __syncthreads();
  am = red[0]; f2 = red[NW];
#pragma unroll
  for (int w = 1; w < NW; ++w) { am = fmaxf(am, red[w]); f2 += red[NW + w]; }
  int ex = 0;
  (void)frexpf(am, &ex);
  const float sT = ldexpf(1.f, 7 - ex), sX = ldexpf(1.f, 7 + ex), inv_sX = ldexpf(1.f, -7 - ex);
  // the wave's rows of T as A operands
  halfx8 th[NS], tl[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const float* p = trow + 16 * s + 8 * h;
    const float4 u0 = *reinterpret_cast<const float4*>(p), u1 = *reinterpret_cast<const float4*>(p + 4);
    const float y[8] = {u0.x * sT, u0.y * sT, u0.z * sT, u0.w * sT, u1.x * sT, u1.y * sT, u1.z * sT, u1.w * sT};
    uintx4 ph, pl;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ph[e] = pack_f16(y[2 * e], y[2 * e + 1]);
      pl[e] = pack_f16_rest(y[2 * e], y[2 * e + 1], ph[e]);
    }
    th[s] = as_halfx8(ph);
    tl[s] = as_halfx8(pl);
  }
  bool unit = false;
  if constexpr (WARM) {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) x[t][v] = Ob[(i0 + 8 * (v / 4) + (v % 4)) * K + j0 + 32 * t] * sX;
  } else {
    const float alpha = f2 * (1.f / K);
    unit = fabsf(alpha - 1.f) <= 1e-5f;
    const float m = unit ? sX : sX / alpha;
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) x[t][v] *= m;
  }

  enum { kEliminate, kTranspose, kConverged };
  int result = kEliminate;
  float prev = 0.f;
#pragma unroll 1
  for (int it = 0; it < kMaxRounds; ++it) {
    // (red and, from the second round on, xr and rt are still being read by slower waves)
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float a0 = x[t][4 * g], a1 = x[t][4 * g + 1], a2 = x[t][4 * g + 2], a3 = x[t][4 * g + 3];
        const int o = (j0 + 32 * t) * LDH + i0 + 8 * g, q = (i0 + 8 * g) * LDH + j0 + 32 * t;
        uint2 ph, pl;
        ph.x = pack_f16(a0, a1); ph.y = pack_f16(a2, a3);
        pl.x = pack_f16_rest(a0, a1, ph.x);
        pl.y = pack_f16_rest(a2, a3, ph.y);
        *reinterpret_cast<uint2*>(xth + o) = ph;
        *reinterpret_cast<uint2*>(xtl + o) = pl;
        xr[q] = uint16_t(ph.x); xr[q + LDH] = uint16_t(ph.x >> 16);
        xr[q + 2 * LDH] = uint16_t(ph.y); xr[q + 3 * LDH] = uint16_t(ph.y >> 16);
      }
    __syncthreads();
    // acc = -2^14 R
    floatx16 acc[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
      if (j0 + 32 * t - ln == i0 - 4 * h) {      // a tile on the diagonal (uniform over the wave)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 8 * (v / 4) + (v % 4) + 4 * h == ln ? -0x1p14f : 0.f;
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const int o = (j0 + 32 * t) * LDH + 16 * s + 8 * h;
        const halfx8 bh = as_halfx8(*reinterpret_cast<const uintx4*>(xth + o));
        const halfx8 bl = as_halfx8(*reinterpret_cast<const uintx4*>(xtl + o));
        acc[t] = CAFEQ_MFMA_F16(tl[s], bh, acc[t]);
        acc[t] = CAFEQ_MFMA_F16(th[s], bl, acc[t]);
        acc[t] = CAFEQ_MFMA_F16(th[s], bh, acc[t]);
      }
    float m = 0.f, q = 0.f;                      // (m passes over a NaN, q does not)
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        m = fmaxf(m, fabsf(acc[t][v]));
        q = fmaf(acc[t][v], acc[t][v], q);
      }
    m = cluster_allmax<64>(m);
    q = wave_sum(q);
    if (lane == 0) { red[wave] = m; red[NW + wave] = q; }
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 pk;
        pk.x = pack_f16(acc[t][4 * g], acc[t][4 * g + 1]);
        pk.y = pack_f16(acc[t][4 * g + 2], acc[t][4 * g + 3]);
        *reinterpret_cast<uint2*>(rt + (j0 + 32 * t) * LDH + i0 + 8 * g) = pk;
      }
    __syncthreads();
    float rmax = red[0], fro2 = red[NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) { rmax = fmaxf(rmax, red[w]); fro2 += red[NW + w]; }
    rmax *= 0x1p-14f;
    fro2 *= 0x1p-28f;
    // R_new = R^2: a contraction at every round, or none to count on (a start outside, a NaN, noise above the bound)
    if (!(fro2 < (WARM ? 0.25f : 9.f)) || (it > 0 && !(fro2 < 0.7f * prev))) break;
    if (K != 32 && unit && it == 0 && rmax <= 2e-6f) { result = kTranspose; break; }
    const bool last = fro2 <= 9e-6f;             // then ||R||_F <= 9e-6 and what the parts lose: 2e-5 is expected
    prev = fro2;
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const halfx8 av = as_halfx8(*reinterpret_cast<const uintx4*>(xr + (i0 - 4 * h + ln) * LDH + 16 * s + 8 * h));
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const halfx8 bv = as_halfx8(*reinterpret_cast<const uintx4*>(rt + (j0 + 32 * t) * LDH + 16 * s + 8 * h));
        acc[t] = CAFEQ_MFMA_F16(av, bv, acc[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) x[t][v] = fmaf(acc[t][v], -0x1p-14f, x[t][v]);
    if (last) { result = kConverged; break; }
  }

  // the step with the exact residual; false: X is not the inverse it was taken for
  auto refine = [&]() __attribute__((always_inline)) {
    float xm = 0.f;
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) xm = fmaxf(xm, fabsf(x[t][v]));
    xm = cluster_allmax<64>(xm);
    // T again, as digits of 2^-ex T: A operands, sixteen contraction indices per lane and step
    __syncthreads();                           // (slower waves are still reading red and the last round's operands)
    if (lane == 0) red[wave] = xm;
    stage_t();
    __syncthreads();
    xm = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) xm = fmaxf(xm, red[w]);
    int exx = 0;
    (void)frexpf(xm, &exx);
    // T X is 2^sh times the sum of the digits' products (x itself carries sX = 2^(7 + ex)); what lies below the digits is
    // 2^(sh - 31) or so of it
    const int sh = exx - 7;
    if (sh > NsShape<K>::kMaxShift) return false;
    const float sd = ldexpf(1.f, -exx);
    intx4 td[4][K / 32];
#pragma unroll
    for (int s = 0; s < K / 32; ++s)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 u = *reinterpret_cast<const float4*>(trow + 32 * s + 16 * h + 4 * g);
        const float sc = ldexpf(1.f, -ex), y[4] = {u.x * sc, u.y * sc, u.z * sc, u.w * sc};
        uint32_t d[4];
        digit_words(y, d);
#pragma unroll
        for (int p = 0; p < 4; ++p) td[p][s][g] = int(d[p]);
      }
    unsigned char* dig = ns_lds;               // [digit][j][LDG]: X^T
    __syncthreads();                           // every wave has its rows of T
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float y[4] = {x[t][4 * g] * sd, x[t][4 * g + 1] * sd, x[t][4 * g + 2] * sd, x[t][4 * g + 3] * sd};
        uint32_t d[4];
        digit_words(y, d);
#pragma unroll
        for (int p = 0; p < 4; ++p)
          *reinterpret_cast<uint32_t*>(dig + (p * K + j0 + 32 * t) * S::LDG + i0 + 8 * g) = d[p];
      }
    __syncthreads();
    // one sum per weight 2^-12, 2^-20, .. 2^-44 (neighbouring matrix instructions then do not depend on each other), each
    // below 2^23 (the first digits are at most 64), taken from the identity largest first: what is left after each is small
    // enough to be exact in float32
    uint2 rp[TPW][4];                          // 2^20 R
    const float rs = ldexpf(1.f, 20 + sh), back = 0x1p-20f;
    float f2 = 0.f;
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      intx16 part[5];
#pragma unroll
      for (int w = 0; w < 5; ++w)
#pragma unroll
        for (int v = 0; v < 16; ++v) part[w][v] = 0;
#pragma unroll
      for (int s = 0; s < K / 32; ++s) {
        intx4 xd[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          xd[q] = *reinterpret_cast<const intx4*>(dig + (q * K + j0 + 32 * t) * S::LDG + 32 * s + 16 * h);
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (p + q < 5) part[p + q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(td[p][s], xd[q], part[p + q], 0, 0, 0);
      }
      const float one = j0 + 32 * t - ln == i0 - 4 * h ? ldexpf(1.f, -sh) : 0.f;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float u[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int v = 4 * g + e;
          u[e] = fmaf(float(part[0][v]), -0x1p-12f, 8 * g + e + 4 * h == ln ? one : 0.f);
          u[e] = fmaf(float(part[1][v]), -0x1p-20f, u[e]);
          u[e] = fmaf(float(part[2][v]), -0x1p-28f, u[e]);
          u[e] = fmaf(float(part[3][v] * 256 + part[4][v]), -0x1p-44f, u[e]) * rs;
          f2 = fmaf(u[e], u[e], f2);
        }
        rp[t][g] = make_uint2(pack_f16(u[0], u[1]), pack_f16(u[2], u[3]));
      }
    }
    f2 = wave_sum(f2);
    if (lane == 0) red[NW + wave] = f2;
    __syncthreads();                           // every wave is done with the digits
    f2 = red[NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) f2 += red[NW + w];
    if (!(f2 * 0x1p-40f <= 4e-10f)) return false;
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) *reinterpret_cast<uint2*>(rt + (j0 + 32 * t) * LDH + i0 + 8 * g) = rp[t][g];
    __syncthreads();
    floatx16 acc[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    // (xr: X before the last round's update; the difference is of third order)
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const halfx8 av = as_halfx8(*reinterpret_cast<const uintx4*>(xr + (i0 - 4 * h + ln) * LDH + 16 * s + 8 * h));
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const halfx8 bv = as_halfx8(*reinterpret_cast<const uintx4*>(rt + (j0 + 32 * t) * LDH + 16 * s + 8 * h));
        acc[t] = CAFEQ_MFMA_F16(av, bv, acc[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) x[t][v] = fmaf(acc[t][v], back, x[t][v]);
    return true;
  };
  if (result == kConverged && !refine()) result = kEliminate;
  if (result == kEliminate) {
    __syncthreads();                             // LDS changes hands
    return false;
  }
  // (an offset of its own: with the one of the warm start's loads their addresses stayed in registers all the way)
  int at = i0 * K + j0;
  asm volatile("" : "+v"(at));
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) Ob[at + (8 * (v / 4) + (v % 4)) * K + 32 * t] = x[t][v] * inv_sX;
  if (status && tid == 0) status[b] = 0;
  return true;
}
__device__ __forceinline__ GjArgs ns_eliminate_args(int K, const float* T, float* Tinv, int* status) {
  GjArgs a;
  a.K = K; a.nz = 0; a.T = T; a.partial = nullptr; a.out = Tinv;
  a.status = status; a.status_stride = 1; a.status_offset = 0;
  return a;
}

}  // namespace cafeq
