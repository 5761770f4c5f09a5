// Loss / gradient pass over blocks of 32 with groups of 32 (symmetric grid): what xform_core.hpp fuses for larger segments, for the
// one geometry whose strip -- 32 lines x one block -- is a single 32 x 32 matrix tile.
//
// What bounds it: vector instructions and their latencies.  The general kernel spends 1800 instructions and 7.5 k cycles on a strip of 16
// values a lane: a ring of operand stages with four barriers a macro-tile, and a gradient whose eight steps one wave of the four takes for all.
// Here a wave needs nobody else from a block's operands to its partial (800 instructions, 4 k cycles; of those the forward product with its
// splits 1.1 k, arg-max 0.5 k, codes and errors 0.9 k, gradient 0.9 k, error's way back 0.5 k):
//   * the workgroup splits the block's operands itself, so that no launch prepares planes or sums of rho (a block's is its norm's
//     square); each wave splitting them for itself, 40 registers of them, cost as much as it saved (12.8 us below);
//   * the gradient's contraction runs over the strip's own 32 lines, staged through LDS by the wave that reads them (adding coefficient x
//     line into 32 x 32 floats of LDS by atomics: 9.3 k cycles, nine a lane);
//   * the half-waves exchange through v_permlane32_swap, the entry of the largest magnitude is found by comparing with the maximum.
// The gradient's operands are split exactly into three bfloat16 parts like the forward transform's, six products: against float64 1.2e-7 to
// 1.8e-7 off where the general kernel's two parts left 2.5e-6 to 6e-6 and sums by records in float32 1.3e-7 to 2.5e-7 (2 % of the launch).
// Measured (MI355X): 256 x 256 8.2 us and 3.6 us for the planes' launch -> 6.1; 1147 x 2880 19.7 and 4.3 -> 11.9 (both
// with two parts; with three 6.4 and, in descent loops, 12.9).  Three workgroups a
// compute unit instead of two 11.5 (but the launch that adds the partials takes longer), four (128 registers, 16 spilled) 13.
//
#include "xform_core.hpp"

namespace cafeq {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// A wave's room in LDS for the gradient: the weights' three parts transposed ([input][line], rows of 80 bytes: a 16-byte read
// of every lane meets no bank twice) and per line arg-max and coefficient; the wave's share of a partial when that leaves.
constexpr int kC32Row = 80, kC32Plane = 32 * kC32Row, kC32Lines = 3 * kC32Plane, kC32Wave = kC32Lines + 32 * 4 + 32 * 4;
static_assert(kC32Wave % 16 == 0 && kC32Wave >= 4096, "rows, and 32 x 32 floats");

// where |z| == a: best = z, j = J + its place (called from the last values to the first: the lowest index stays).  Comparisons four
// side by side, as in argmax4: a mask is read two instructions later at the earliest.
template <int J>
__device__ __forceinline__ void equal4(float& best, int& j, const float a, const float z0, const float z1, const float z2, const float z3) {
  uint64_t m0, m1, m2, m3;
  asm("v_cmp_eq_f32_e64 %5, |%10|, %6\n\t"
      "v_cmp_eq_f32_e64 %4, |%9|, %6\n\t"
      "v_cmp_eq_f32_e64 %3, |%8|, %6\n\t"
      "v_cmp_eq_f32_e64 %2, |%7|, %6\n\t"
      "v_cndmask_b32_e64 %0, %0, %10, %5\n\t"
      "v_cndmask_b32_e64 %1, %1, %14, %5\n\t"
      "v_cndmask_b32_e64 %0, %0, %9, %4\n\t"
      "v_cndmask_b32_e64 %1, %1, %13, %4\n\t"
      "v_cndmask_b32_e64 %0, %0, %8, %3\n\t"
      "v_cndmask_b32_e64 %1, %1, %12, %3\n\t"
      "v_cndmask_b32_e64 %0, %0, %7, %2\n\t"
      "v_cndmask_b32_e64 %1, %1, %11, %2"
      : "+&v"(best), "+&v"(j), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
      : "v"(a), "v"(z0), "v"(z1), "v"(z2), "v"(z3), "n"(J), "n"(J + 1), "n"(J + 2), "n"(J + 3));
}
// (lower half's x, upper half's x), in every lane
struct Halves { uint32_t lo, hi; };
__device__ __forceinline__ Halves halves(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return Halves{r[0], r[1]};
}

template <int AXIS, bool GRAD>
__global__ __launch_bounds__(kThreads, 3) void core32_kernel(const CoreParams p) {
  constexpr int K = 32;
  __shared__ __align__(16) unsigned char room[GRAD ? kNW : 1][GRAD ? kC32Wave : 16];
  __shared__ __align__(16) unsigned char planes[5 * 2048];   // [forward hi, mid, lo; inverse hi, mid][out][32 inputs]
  __shared__ float hred[kNW][8], rsum[kNW];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, h = lane >> 5;
  // contiguous ranges; consecutive ones on the same XCD
  uint32_t w = blockIdx.x;
  if ((p.nwg & 7) == 0) w = (blockIdx.x & 7) * (uint32_t(p.nwg) >> 3) + (blockIdx.x >> 3);
  int64_t mt0, mt1;
  if (p.n_mt == p.nwg) {
    mt0 = w; mt1 = w + 1;
  } else {
    mt0 = chunk_begin(w, p.n_mt, p.nwg); mt1 = chunk_begin(w + 1, p.n_mt, p.nwg);
  }
  if (mt0 >= mt1) return;
  const int mt_per_seg = int(p.mt_per_seg);
  int seg, mis;
  if (uint64_t(mt0) < (uint64_t(1) << 32)) {
    seg = int(uint32_t(mt0) / uint32_t(mt_per_seg));
  } else {
    seg = int(mt0 / p.mt_per_seg);
  }
  mis = int(mt0 - int64_t(seg) * mt_per_seg);
  int left = int(mt1 - mt0);

  // element j(f) = 8 (f / 4) + 4 h + f % 4 of the lane's line of a macro-tile
  auto load_w = [&](int seg_, int mis_, float (&x)[16]) __attribute__((always_inline)) {
    const int64_t line = int64_t(mis_) * kMacroLines + wave * kStripLines + ln;
    const int64_t lc = line < p.nlines ? line : p.nlines - 1;
    if (AXIS == CAFEQ_AXIS_COL) {
      const int64_t at = lc * p.ld + int64_t(seg_) * K + 4 * h;
      if (p.dtype == CAFEQ_F32) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float4 v = *reinterpret_cast<const float4*>(static_cast<const float*>(p.W) + at + 8 * c);
          x[4 * c] = v.x; x[4 * c + 1] = v.y; x[4 * c + 2] = v.z; x[4 * c + 3] = v.w;
        }
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float4 v = load4(static_cast<const uint16_t*>(p.W) + at + 8 * c);
          x[4 * c] = v.x; x[4 * c + 1] = v.y; x[4 * c + 2] = v.z; x[4 * c + 3] = v.w;
        }
      }
    } else {
      const uint32_t loff = uint32_t(int64_t(4 * h) * p.ld + lc);   // (uniform row pointer, 32-bit lane offset)
      const int64_t at = int64_t(seg_) * K * p.ld;
      if (p.dtype == CAFEQ_F32) {
        const float* rp = static_cast<const float*>(p.W) + at;
#pragma unroll
        for (int f = 0; f < 16; ++f) x[f] = (rp + (8 * (f / 4) + f % 4) * p.ld)[loff];
      } else {
        const uint16_t* rp = static_cast<const uint16_t*>(p.W) + at;
#pragma unroll
        for (int f = 0; f < 16; ++f) x[f] = bf16_bits_to_f32((rp + (8 * (f / 4) + f % 4) * p.ld)[loff]);
      }
    }
  };

  float rg = 0.f;               // kLossSur: sum of the block's rho
  // three (or two) bfloat16 parts of eight values
  auto split3 = [](const float* x, bf16x8& hi, bf16x8& mid, bf16x8& lo) __attribute__((always_inline)) {
    uint32_t a[4], b[4], c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = pack_bf16(x[2 * i], x[2 * i + 1]);
      const float r0 = x[2 * i] - bf16_lo_f32(a[i]), r1 = x[2 * i + 1] - bf16_hi_f32(a[i]);
      b[i] = pack_bf16(r0, r1);
      c[i] = pack_bf16(r0 - bf16_lo_f32(b[i]), r1 - bf16_hi_f32(b[i]));
    }
    hi = as_bf16x8(a[0], a[1], a[2], a[3]); mid = as_bf16x8(b[0], b[1], b[2], b[3]); lo = as_bf16x8(c[0], c[1], c[2], c[3]);
  };
  auto split3q = [](const float (&x)[4], uint2& hi, uint2& mid, uint2& lo) __attribute__((always_inline)) {
    hi = make_uint2(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]));
    const float r0 = x[0] - bf16_lo_f32(hi.x), r1 = x[1] - bf16_hi_f32(hi.x), r2 = x[2] - bf16_lo_f32(hi.y), r3 = x[3] - bf16_hi_f32(hi.y);
    mid = make_uint2(pack_bf16(r0, r1), pack_bf16(r2, r3));
    lo = make_uint2(pack_bf16(r0 - bf16_lo_f32(mid.x), r1 - bf16_hi_f32(mid.x)), pack_bf16(r2 - bf16_lo_f32(mid.y), r3 - bf16_hi_f32(mid.y)));
  };
  auto split2 = [](const float* x, bf16x8& hi, bf16x8& mid) __attribute__((always_inline)) {
    uint32_t a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = pack_bf16(x[2 * i], x[2 * i + 1]);
      b[i] = pack_bf16(x[2 * i] - bf16_lo_f32(a[i]), x[2 * i + 1] - bf16_hi_f32(a[i]));
    }
    hi = as_bf16x8(a[0], a[1], a[2], a[3]); mid = as_bf16x8(b[0], b[1], b[2], b[3]);
  };
  auto block_of = [&](int seg_) { return AXIS == CAFEQ_AXIS_ROW && p.rep != 1 ? int(uint32_t(seg_) / uint32_t(p.rep)) : seg_; };

  float s_l2 = 0.f, s_errz = 0.f, s_wsq = 0.f, s_sur = 0.f, s_va2 = 0.f;
  float m_ref = -INFINITY;      // kLossLse: reference of this wave's exponentials
  const bool lse = p.loss_kind == kLossLse;
  floatx16 gt;                  // element [row 8 (v / 4) + 4 h + v % 4][input ln] of the block's gradient, this wave's lines
#pragma unroll
  for (int v = 0; v < 16; ++v) gt[v] = 0.f;
  unsigned char* wst = room[GRAD ? wave : 0];
  uint32_t* jst = reinterpret_cast<uint32_t*>(wst + (GRAD ? kC32Lines : 0));         // arg-max | coefficient's third part << 16
  uint32_t* cfp = reinterpret_cast<uint32_t*>(wst + (GRAD ? kC32Lines + 128 : 0));   // its first | its second << 16

  float x[16], xn[16] = {};
  load_w(seg, mis, x);
  int have = -1;                // the block whose operands are in LDS
  // A operands: row ln, chunk 2 c + h
  const int swz = (ln >> 2) & 3, aoff0 = ln * 64 + ((h ^ swz) << 4), aoff1 = ln * 64 + (((2 + h) ^ swz) << 4);
  bool more, whole;
  int last_seg;
  do {                          // (one exit, at the end: with a way out behind the partial the compiler left out the copy of xn there)
    more = left > 1;
    int nseg = seg, nmis = mis + 1;
    if (nmis == mt_per_seg) { nmis = 0; ++nseg; }
    const int bid = block_of(seg);
    if (bid != have) {
      // the workgroup splits the block's operands, four inputs of one output row a thread: [out][in], T and T^-1 read transposed along columns
      const int out = AXIS == CAFEQ_AXIS_COL ? tid & 31 : tid >> 3, wq = AXIS == CAFEQ_AXIS_COL ? tid >> 5 : tid & 7;
      const float *tf = p.Tfwd + size_t(bid) * (K * K), *tb = p.Tback + size_t(bid) * (K * K);
      float t[4], u[4];
      if (AXIS == CAFEQ_AXIS_COL) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { t[e] = tf[(4 * wq + e) * K + out]; u[e] = tb[(4 * wq + e) * K + out]; }
      } else {
        const float4 a = *reinterpret_cast<const float4*>(tf + 4 * tid), b = *reinterpret_cast<const float4*>(tb + 4 * tid);
        t[0] = a.x; t[1] = a.y; t[2] = a.z; t[3] = a.w;
        u[0] = b.x; u[1] = b.y; u[2] = b.z; u[3] = b.w;
      }
      if (have >= 0) __syncthreads();                  // (the block before is still being read)
      // quad wq: inputs 16 c + 8 u + 4 h + e, in chunk 2 c + h of the row's four (swizzled)
      unsigned char* at = planes + out * 64 + (((wq >> 2) * 2 + (wq & 1)) ^ ((out >> 2) & 3)) * 16 + ((wq >> 1) & 1) * 8;
      uint2 p0, p1, p2;
      split3q(t, p0, p1, p2);
      *reinterpret_cast<uint2*>(at) = p0;
      *reinterpret_cast<uint2*>(at + 2048) = p1;
      *reinterpret_cast<uint2*>(at + 4096) = p2;
      split3q(u, p0, p1, p2);
      *reinterpret_cast<uint2*>(at + 6144) = p0;
      *reinterpret_cast<uint2*>(at + 8192) = p1;
      if (!lse) {
        const double r = __builtin_fma(double(u[0]), double(u[0]), double(u[1]) * u[1]) + __builtin_fma(double(u[2]), double(u[2]), double(u[3]) * u[3]);
        const float rw = wave_sum(float(r));
        if (lane == 0) rsum[wave] = rw;
      }
      __syncthreads();
      if (!lse) rg = (rsum[0] + rsum[1]) + (rsum[2] + rsum[3]);
      have = bid;
    }
    if (more) load_w(nseg, nmis, xn);
    const int64_t line = int64_t(mis) * kMacroLines + wave * kStripLines + ln;
    const bool valid = line < p.nlines;
    if (!valid) {
#pragma unroll
      for (int f = 0; f < 16; ++f) x[f] = 0.f;
    }
    float wsq = 0.f;
#pragma unroll
    for (int f = 0; f < 16; ++f) wsq = fmaf(x[f], x[f], wsq);

    if (!lse && p.rG_out && tid == 0) p.rG_out[seg] = rg;   // (a segment's workgroups write the same)

    // ---- Z: six products, smallest terms first
    floatx16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      bf16x8 bh, bm, bl;
      split3(x + 8 * c, bh, bm, bl);
      const unsigned char* ap = planes + (c == 0 ? aoff0 : aoff1);
      const bf16x8 fh = as_bf16x8(*reinterpret_cast<const uintx4*>(ap)), fm = as_bf16x8(*reinterpret_cast<const uintx4*>(ap + 2048)),
                   fl = as_bf16x8(*reinterpret_cast<const uintx4*>(ap + 4096));
      if constexpr (GRAD) {
        const uintx4 uh = __builtin_bit_cast(uintx4, bh), um = __builtin_bit_cast(uintx4, bm), ul = __builtin_bit_cast(uintx4, bl);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          unsigned char* at = wst + (16 * c + 8 * (i / 2) + 4 * h + 2 * (i % 2)) * kC32Row + 2 * ln;
          *reinterpret_cast<uint16_t*>(at) = uint16_t(uh[i]);
          *reinterpret_cast<uint16_t*>(at + kC32Row) = uint16_t(uh[i] >> 16);
          *reinterpret_cast<uint16_t*>(at + kC32Plane) = uint16_t(um[i]);
          *reinterpret_cast<uint16_t*>(at + kC32Plane + kC32Row) = uint16_t(um[i] >> 16);
          *reinterpret_cast<uint16_t*>(at + 2 * kC32Plane) = uint16_t(ul[i]);
          *reinterpret_cast<uint16_t*>(at + 2 * kC32Plane + kC32Row) = uint16_t(ul[i] >> 16);
        }
      }
      z = CAFEQ_MFMA_BF16(fl, bh, z);
      z = CAFEQ_MFMA_BF16(fh, bl, z);
      z = CAFEQ_MFMA_BF16(fm, bm, z);
      z = CAFEQ_MFMA_BF16(fm, bh, z);
      z = CAFEQ_MFMA_BF16(fh, bm, z);
      z = CAFEQ_MFMA_BF16(fh, bh, z);
    }
    s_wsq += wsq;

    // ---- the group's largest magnitude, the entry that has it (of several the lowest), codes and errors
    float a = -1.f;
#pragma unroll
    for (int f = 0; f < 16; ++f) a = fmaxf(a, fabsf(z[f]));
    float zs = 0.f;
    int j = 4;                  // (of a group without a number the entry is 4, as in the general kernel)
    equal4<24>(zs, j, a, z[12], z[13], z[14], z[15]);
    equal4<16>(zs, j, a, z[8], z[9], z[10], z[11]);
    equal4<8>(zs, j, a, z[4], z[5], z[6], z[7]);
    equal4<0>(zs, j, a, z[0], z[1], z[2], z[3]);
    j += 4 * h;
    {
      const Halves zz = halves(__float_as_uint(zs)), jj = halves(uint32_t(j));
      const float z0 = __uint_as_float(zz.lo), z1 = __uint_as_float(zz.hi);
      const bool up = fabsf(z1) > fabsf(z0) || (fabsf(z1) == fabsf(z0) && int(jj.hi) < int(jj.lo));
      zs = up ? z1 : z0;
      j = int(up ? jj.hi : jj.lo);
    }
    a = fabsf(zs);
    if (p.rec && valid && h == 0) p.rec[int64_t(seg) * p.nlines + line] = make_float2(zs, __int_as_float(j));
    const float inv = grid_inv(a, p.grid.qmax), s = grid_scale(a, p.grid.qmax);
    if (p.scales && valid && h == 0) p.scales[AXIS == CAFEQ_AXIS_COL ? line * p.nseg + seg : int64_t(seg) * p.cols + line] = s;
    float err[16];
    uint32_t qpk[4];
#pragma unroll
    for (int f4 = 0; f4 < 4; ++f4) {
      float q[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = z[4 * f4 + e];
        q[e] = grid_code(v, inv, p.grid);
        const float er = __fmul_rn(q[e], s) - v;
        s_errz = fmaf(er, er, s_errz);
        err[4 * f4 + e] = er;
      }
      qpk[f4] = p.codes ? pack4(q[0], q[1], q[2], q[3]) : 0u;
    }
    if (AXIS == CAFEQ_AXIS_COL && p.codes) {
      // 16 of the group's 32 codes each: a lane holds every other four of them, the half-waves exchange two.  (In stores of 4 bytes a lane the codes
      // of 36864 x 4608 took the call 445 us, now 411; the general kernel 436.)
      const auto a02 = __builtin_amdgcn_permlane32_swap(qpk[0], qpk[2], false, false), a13 = __builtin_amdgcn_permlane32_swap(qpk[1], qpk[3], false, false);
      const uintx4 c = {a02[0], a02[1], a13[0], a13[1]};
      if (valid) *reinterpret_cast<uintx4*>(p.codes + line * p.cols + int64_t(seg) * K + 16 * h) = c;
    }
    if (AXIS == CAFEQ_AXIS_ROW && p.codes && valid) {
      const int64_t ax0 = int64_t(seg) * K;
      const uint32_t loff = uint32_t(4 * h) * uint32_t(p.cols) + uint32_t(line);
#pragma unroll
      for (int f4 = 0; f4 < 4; ++f4)
#pragma unroll
        for (int e = 0; e < 4; ++e) (p.codes + (ax0 + 8 * f4 + e) * p.cols)[loff] = int8_t(qpk[f4] >> (8 * e));
    }
    if (h == 0) s_va2 = fmaf(a, a, s_va2);
    float coef;
    if (!lse) {
      if (h == 0) s_sur = fmaf(a * a, rg, s_sur);
      coef = 2.f * p.beta * rg * zs;
    } else {
      const float mx = cluster_allmax<64>(valid ? a : 0.f);
      if (mx > m_ref) {                                 // (uniform)
        const float sc = __expf(p.lse_t * (m_ref - mx));
        s_sur *= sc;
        if constexpr (GRAD) {
#pragma unroll
          for (int v = 0; v < 16; ++v) gt[v] *= sc;
        }
        m_ref = mx;
      }
      const float e = valid ? __expf(p.lse_t * (a - m_ref)) : 0.f;
      if (h == 0) s_sur += e;
      coef = zs < 0.f ? -e : e;
    }

    // ---- the gradient: G[j][m] += sum over the strip's lines of S[line][j] W[line][m], S's parts built from (arg-max, coefficient)
    if constexpr (GRAD) {
      if (h == 0) {
        // coefficient in three bfloat16 parts
        const uint32_t c0 = pack_bf16(coef, 0.f) & 0xFFFFu;
        const float r0 = coef - bf16_lo_f32(c0);
        const uint32_t c1 = pack_bf16(r0, 0.f) & 0xFFFFu, c2 = pack_bf16(r0 - bf16_lo_f32(c1), 0.f);
        jst[ln] = uint32_t(j) | c2 << 16;
        cfp[ln] = c0 | c1 << 16;
      }
      // (within the wave alone: its LDS instructions run in order)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int l0 = 16 * c + 8 * h;
        const uintx4 j0 = *reinterpret_cast<const uintx4*>(jst + l0), j1 = *reinterpret_cast<const uintx4*>(jst + l0 + 4);
        const uintx4 c0 = *reinterpret_cast<const uintx4*>(cfp + l0), c1 = *reinterpret_cast<const uintx4*>(cfp + l0 + 4);
        const unsigned char* wrow = wst + ln * kC32Row + 2 * l0;
        const bf16x8 bh = as_bf16x8(*reinterpret_cast<const uintx4*>(wrow)), bm = as_bf16x8(*reinterpret_cast<const uintx4*>(wrow + kC32Plane)),
                     bl = as_bf16x8(*reinterpret_cast<const uintx4*>(wrow + 2 * kC32Plane));
        uint32_t sel[8], third[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t jv = e < 4 ? j0[e] : j1[e - 4];
          const bool mine = (jv & 0xFFFFu) == uint32_t(ln);
          sel[e] = mine ? (e < 4 ? c0[e] : c1[e - 4]) : 0u;
          third[e] = mine ? jv : 0u;
        }
        uintx4 sh, sm, sl;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sh[e] = __builtin_amdgcn_perm(sel[2 * e + 1], sel[2 * e], 0x05040100u);
          sm[e] = __builtin_amdgcn_perm(sel[2 * e + 1], sel[2 * e], 0x07060302u);
          sl[e] = __builtin_amdgcn_perm(third[2 * e + 1], third[2 * e], 0x07060302u);
        }
        // six products, smallest terms first
        gt = CAFEQ_MFMA_BF16(as_bf16x8(sl), bh, gt);
        gt = CAFEQ_MFMA_BF16(as_bf16x8(sh), bl, gt);
        gt = CAFEQ_MFMA_BF16(as_bf16x8(sm), bm, gt);
        gt = CAFEQ_MFMA_BF16(as_bf16x8(sm), bh, gt);
        gt = CAFEQ_MFMA_BF16(as_bf16x8(sh), bm, gt);
        gt = CAFEQ_MFMA_BF16(as_bf16x8(sh), bh, gt);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }

    // ---- D = T^-1 E: three products
    floatx16 d;
#pragma unroll
    for (int v = 0; v < 16; ++v) d[v] = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      bf16x8 eh, em;
      split2(err + 8 * c, eh, em);
      const unsigned char* ap = planes + 6144 + (c == 0 ? aoff0 : aoff1);
      const bf16x8 ih = as_bf16x8(*reinterpret_cast<const uintx4*>(ap)), im = as_bf16x8(*reinterpret_cast<const uintx4*>(ap + 2048));
      d = CAFEQ_MFMA_BF16(im, eh, d);
      d = CAFEQ_MFMA_BF16(ih, em, d);
      d = CAFEQ_MFMA_BF16(ih, eh, d);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) s_l2 = fmaf(d[v], d[v], s_l2);

    if (!more || nseg != seg) {
      // ---- the partial of this (workgroup, segment): waves added in their order
      const int64_t slot = int64_t(w) + seg;
      const float v0 = wave_sum(s_l2), v1 = wave_sum(s_errz), v2 = wave_sum(s_wsq), v3 = wave_sum(s_sur), v4 = wave_sum(s_va2);
      if constexpr (GRAD) {
        // (lane's four entries side by side: [quad of v][lane])
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(wst + (q * 64 + lane) * 16) = make_float4(gt[4 * q], gt[4 * q + 1], gt[4 * q + 2], gt[4 * q + 3]);
      }
      if (lane < 6) hred[wave][lane] = lane == 0 ? v0 : lane == 1 ? v1 : lane == 2 ? v2 : lane == 3 ? v3 : lane == 4 ? m_ref : v4;
      __syncthreads();
      float mm = hred[0][4], sc[kNW];
#pragma unroll
      for (int k = 1; k < kNW; ++k) mm = fmaxf(mm, hred[k][4]);
#pragma unroll
      for (int k = 0; k < kNW; ++k) sc[k] = lse ? (hred[k][4] == mm ? 1.f : __expf(p.lse_t * (hred[k][4] - mm))) : 1.f;
      if (tid < kHdrVa2 + 1) {
        const int src = tid < 4 ? tid : 5;
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < kNW; ++k) t += hred[k][src] * (tid == kHdrSur ? sc[k] : 1.f);
        if (tid == kHdrMref) t = mm;
        if (tid > kHdrMref && tid < kHdrVa2) t = 0.f;
        p.slot_hdr[slot * kHdrFloats + tid] = t;
      }
      if constexpr (GRAD) {
        // entry [8 q + 4 h + e][ln]: quad q of lane 32 h + ln, that is wave q's and this lane's
        floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kNW; ++k) {
          const float4 t = *reinterpret_cast<const float4*>(room[GRAD ? k : 0] + tid * 16);
          o[0] += sc[k] * t.x; o[1] += sc[k] * t.y; o[2] += sc[k] * t.z; o[3] += sc[k] * t.w;
        }
        float* dst = p.slot_grad + slot * int64_t(K * K) + (8 * wave + 4 * h) * K + ln;
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e * K] = o[e];
      }
      __syncthreads();
#pragma unroll
      for (int v = 0; v < 16; ++v) gt[v] = 0.f;
      s_l2 = s_errz = s_wsq = s_sur = s_va2 = 0.f;
      m_ref = -INFINITY;
    }
#pragma unroll
    for (int f = 0; f < 16; ++f) x[f] = xn[f];
    last_seg = seg;
    whole = nmis == 0;
    seg = nseg;
    mis = nmis;
    --left;
  } while (more);
  // a range that ends with its segment leaves the header behind its last one to nobody (workgroup w + 1 begins a segment
  // further): it must read as empty
  if (whole && tid < kHdrFloats)
    p.slot_hdr[(int64_t(w) + last_seg + 1) * kHdrFloats + tid] = tid == kHdrMref ? -INFINITY : 0.f;
}

}  // namespace

int launch_core32(int axis, const CoreParams& p, hipStream_t st) {
  if (!p.do_inverse || !p.Tfwd || !p.Tback || !p.slot_hdr || p.Zout || p.longg || p.asym || (p.do_grad && !p.slot_grad)) return CAFEQ_ERR_INVALID_ARG;
  const dim3 grid(unsigned(p.nwg)), block(kThreads);
  if (axis == CAFEQ_AXIS_COL) {
    if (p.do_grad) hipLaunchKernelGGL((core32_kernel<CAFEQ_AXIS_COL, true>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((core32_kernel<CAFEQ_AXIS_COL, false>), grid, block, 0, st, p);
  } else {
    if (p.do_grad) hipLaunchKernelGGL((core32_kernel<CAFEQ_AXIS_ROW, true>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((core32_kernel<CAFEQ_AXIS_ROW, false>), grid, block, 0, st, p);
  }
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}

}  // namespace cafeq
