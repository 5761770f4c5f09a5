// Fused transform / quantize / inverse-transform pass for blocks of 256 and groups up to 256 (the paths of xform_core.hpp
// for the symmetric grid; longer groups and the min/max grid stay there).
//
// A strip of 32 lines x one block is the work of TWO waves, 128 outputs each.  One wave holding all 256 (xform_core.hpp)
// needs 128 accumulators, 128 errors and 128 weights a lane: one wave per SIMD, 184 to 288 bytes of scratch a lane, and nothing
// that runs beside its matrix instructions.  With half of each a wave fits 256 registers without scratch, and the two waves of a strip
// share a SIMD: one splits operands or quantizes while the other feeds the matrix pipe.
//
// What a half needs of the other goes through LDS: the operands of the contraction.  A stage is 32 contraction indices; the wave
// that holds them (weights going forward, errors going back) splits them into one to three bfloat16 parts in the operand's own lane order,
// 16 bytes a lane and part, one stage ahead, and both waves read them back.  The transform's planes (bfloat16, three parts going
// forward, two going back) stream through 96 KB of LDS, two stages of 48 KB and then three of 32, one barrier a stage.
//
// Arithmetic: the bfloat16 parts of xform_core.hpp, unscaled: every operand keeps float32's range and going forward all of its 24 bits,
// however far it lies below the rest of its line or block, and a transform that only moves weights moves them exactly.  (Two and three
// float16 parts, scaled per line and block, are a third fewer products, but hold nothing below 2^-39 of the largest and all bits only
// down to 2^-14 of it.)  Forward: six products, a stage's in a sum of their own, so that one rounding in
// eight is at the size of the result.  Z against float64, in units of its line's root mean square, this / all products into one sum:
// rotations, 5 and 50 % off them 9.1e-8 / 2.4e-7; identities 1e-4 off 1.0e-7 / 1.6e-7, 1e-2 off 9.9e-8 / 1.9e-7; identities and
// permutations exact.  Back: two parts each, three products.
// Adaptive rounding multiplies by what the correction adds to the identity.
//
// Bound: issue of matrix instructions, 48 a stage and wave going forward and 24 going back, two waves a SIMD, against 30 (20) KB of
// operands read a wave.  9B-shaped (V, O) pair, groups of 64, loss passes 56 + 110 -> 40 + 75 us (one wave per strip, xform_core.hpp,
// before; on float16 parts 37 + 66); the corrected weights' codes 47 + 80 -> 34 + 57.
#include "gj_panel.hpp"   // StaticFor
#include "xform_launch.hpp"

namespace cafeq {
namespace {

constexpr int kXhK = 256, kXhWaves = 8, kXhThreads = kXhWaves * 64;
constexpr int kXhPlane = kXhK * 64, kXhFwd = kFwdPlanes * kXhPlane, kXhBack = kInvPlanes * kXhPlane;   // bytes: a part of a stage, stages
constexpr int kXhRing = 2 * kXhFwd;
static_assert(kXhRing == 3 * kXhBack, "two stages going forward, three going back");
constexpr int kXhSlot = 4 * 2 * 3 * 1024;                                   // operands of a stage: [strip][step][part][lane][16 B]
constexpr int kXhOpnd = kXhRing, kXhXch = kXhOpnd + 2 * kXhSlot;            // LDS offsets
constexpr int kXhHdr = kXhXch + 2 * 256 * 4;
constexpr int kXhLds = kXhHdr + (kXhWaves * kHdrFloats + kXhWaves) * 4;
// Where stage s lies.  Going forward in halves of the ring, stage 0 in the second and stage 7 in the first; going back in thirds, stage 0 in
// the last, which stage 7 of the way there does not touch, and stage 7 in the first, which stage 0 of the next way there does not.
constexpr int fwd_at(int s) { return ((s + 1) & 1) * kXhFwd; }
constexpr int back_at(int s) { return (s + 2) % 3 * kXhBack; }
static_assert(kXhLds <= 160 * 1024, "one workgroup per compute unit");
static_assert(kMacroLines == 4 * 32, "four strips a workgroup");

// What a launch does: Z alone; a loss call (errors, inverse transform, partial sums); codes and scales of corrected weights
// (adaptive rounding), whose transform is the identity plus a small correction: the planes hold the correction alone, and
// the weights themselves are added to its product
enum XhMode { kXhApply, kXhLoss, kXhCorrect };
// B16: bfloat16 weights, one part themselves: the other two are zeros, and without them a forward stage is 24 matrix instructions
// instead of 48 with the same sums.  Loss pass of 2304 x 9216, groups of 256, with its gradient: 420 -> 403 us a call; (V, O) pair of
// d_model 3584, groups of 64: 312 -> 296; codes of 36864 x 4608, groups of 128: 913 -> 789.
template <int G, int AXIS, XhMode MODE, bool B16>
__global__ __launch_bounds__(kXhThreads, 2) void xform256_kernel(const CoreParams p) {
  constexpr bool INV = MODE == kXhLoss;
  constexpr int K = kXhK, KT = 4, NST = 8;           // tiles of a wave, stages of a block
  constexpr int WP = B16 ? 1 : 3;                    // parts of a weight
  static_assert(MODE != kXhCorrect || !B16, "adaptive rounding works on float32");
  constexpr int TPG = G >= 128 ? 4 : G / 32;         // tiles of one of the wave's groups
  constexpr int NG = 4 / TPG;                        // groups of a wave (G = 256: its half of the one)
  constexpr int NGS = G == 256 ? 1 : 2 * NG;         // groups of a segment
  extern __shared__ __align__(16) unsigned char smem[];
  float* zsg = reinterpret_cast<float*>(smem + kXhXch);       // (G = 256) [2 halves][128 lines]: largest transformed weight
  int* zix = reinterpret_cast<int*>(zsg + 256);               // and its index
  float* hred = reinterpret_cast<float*>(smem + kXhHdr);      // [8][kHdrFloats]
  float* wvm = hred + kXhWaves * kHdrFloats;                  // [8]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int strip = wave & 3, half = wave >> 2;      // (waves i and i + 4 share a SIMD)
  const int ln = lane & 31, h = lane >> 5;
  const int mine = half * 128 + strip * 32 + ln, other = mine ^ 128;

  // contiguous ranges of macro-tiles, consecutive ones behind one L2, as in xform_core.hpp
  int64_t w = blockIdx.x;
  if ((p.nwg & 7) == 0) w = int64_t(blockIdx.x & 7) * (p.nwg >> 3) + (blockIdx.x >> 3);
  const int64_t mt0 = chunk_begin(w, p.n_mt, p.nwg), mt1 = chunk_begin(w + 1, p.n_mt, p.nwg);
  if (mt0 >= mt1) return;
  const int mt_per_seg = int(p.mt_per_seg);
  int seg = int(mt0 / p.mt_per_seg), mis = int(mt0 - int64_t(seg) * p.mt_per_seg), cur_seg = seg;
  auto blk_id = [&](int sg) { return AXIS == CAFEQ_AXIS_ROW && p.rep != 1 ? sg / p.rep : sg; };
  int cb = blk_id(seg);

  // stage s of block b to LDS address `to`, asynchronously (opaque to the compiler, which would otherwise drain it before every LDS read)
  const uint32_t voff = uint32_t(tid) * 16u;
  constexpr int NFB = kXhBack / 16 / kXhThreads;      // requests of a wave and stage, going back
  auto dma = [&](const uint16_t* base, int bytes, int b, int s, int to) __attribute__((always_inline)) {
    const unsigned char* src = reinterpret_cast<const unsigned char*>(base) + (int64_t(b) * NST + s) * bytes;
    const uint32_t at = uint32_t(to) + uint32_t(wave) * 1024u;
#pragma unroll
    for (int i = 0; i < bytes / (16 * kXhThreads); ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(at + uint32_t(i) * (kXhThreads * 16u)), "v"(voff), "s"(src + i * (kXhThreads * 16)) : "memory");
  };

  // The wave's weights: element f is index 128 half + 8 (f / 4) + 4 h + f % 4 of the lane's line; steps [c0, c1) of eight indices.
  // (lines past the matrix read its last one)
  float wreg[64];
  constexpr int NWL = AXIS == CAFEQ_AXIS_COL ? 1 : 4;         // requests of a step
  auto load_w = [&](int sg, int ms, int c0, int c1) __attribute__((always_inline)) {
    int64_t line = int64_t(ms) * kMacroLines + strip * kStripLines + ln;
    if (line >= p.nlines) line = p.nlines - 1;
    const int64_t ax0 = int64_t(sg) * K + 128 * half;
    if constexpr (AXIS == CAFEQ_AXIS_COL) {
      const int64_t at = line * p.ld + ax0 + 4 * h;
#pragma unroll
      for (int c = c0; c < c1; ++c) {
        const float4 v = B16 ? load4(static_cast<const uint16_t*>(p.W) + at + 8 * c) : load4(static_cast<const float*>(p.W) + at + 8 * c);
        wreg[4 * c] = v.x; wreg[4 * c + 1] = v.y; wreg[4 * c + 2] = v.z; wreg[4 * c + 3] = v.w;
      }
    } else {
      const uint32_t loff = uint32_t(int64_t(4 * h) * p.ld + line);
      if constexpr (!B16) {
        const float* rp = static_cast<const float*>(p.W) + (ax0 + 8 * c0) * p.ld;
#pragma unroll
        for (int c = c0; c < c1; ++c) {
#pragma unroll
          for (int e = 0; e < 4; ++e) { wreg[4 * c + e] = rp[loff]; rp += p.ld; }
          rp += 4 * p.ld;
        }
      } else {
        const uint16_t* rp = static_cast<const uint16_t*>(p.W) + (ax0 + 8 * c0) * p.ld;
#pragma unroll
        for (int c = c0; c < c1; ++c) {
#pragma unroll
          for (int e = 0; e < 4; ++e) { wreg[4 * c + e] = bf16_bits_to_f32(rp[loff]); rp += p.ld; }
          rp += 4 * p.ld;
        }
      }
    }
  };
  // sixteen values of a stage (tile s % 4 of the wave that holds it) into the operand slot of stage s
  auto put = [&](auto parts, const float* x, int s) __attribute__((always_inline)) {
    constexpr int NP = decltype(parts)::value;
    unsigned char* at = smem + kXhOpnd + (s & 1) * kXhSlot + strip * (kXhSlot / 4) + lane * 16;
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {
      uintx4 u[NP];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float y0 = x[8 * c2 + 2 * i], y1 = x[8 * c2 + 2 * i + 1];
        asm volatile("" : "+v"(y0), "+v"(y1));       // (not ahead of the branch that this stands in: no registers there)
        // (of an infinity the other parts are not a number, and so is all that it meets)
        if constexpr (NP == 1) { y0 = fmaf(0.f, y0, y0); y1 = fmaf(0.f, y1, y1); }
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) {
          u[pl][i] = pack_bf16(y0, y1);
          y0 -= bf16_lo_f32(u[pl][i]); y1 -= bf16_hi_f32(u[pl][i]);
        }
      }
#pragma unroll
      for (int pl = 0; pl < NP; ++pl) *reinterpret_cast<uintx4*>(at + (c2 * 3 + pl) * 1024) = u[pl];
    }
  };
  // the products of a stage whose planes lie at `at`: the wave's four tiles of 32 outputs, two steps of 16 contraction indices; `between`
  // runs once the first step's operands are requested
  const int swz = (ln >> 2) & 3;
  const int ao[2] = {ln * 64 + ((h ^ swz) << 4), ln * 64 + (((2 + h) ^ swz) << 4)};
  auto products = [&](auto ahead, floatx16 (&c)[KT], floatx16& late, int at, int s, auto&& between) __attribute__((always_inline)) {
    constexpr bool FWD = decltype(ahead)::value;
    constexpr int NP = FWD ? WP : 2, XP = FWD ? kFwdPlanes : kInvPlanes;   // parts of the weights (errors), of the transform
    const unsigned char* a = smem + at + half * (128 * 64);
    const unsigned char* b = smem + kXhOpnd + (s & 1) * kXhSlot + strip * (kXhSlot / 4) + lane * 16;
    bf16x8 y[2][NP], x[2][XP];                       // x: [step]
    auto read = [&](int i) {
#pragma unroll
      for (int pl = 0; pl < XP; ++pl)
        x[i % 2][pl] = as_bf16x8(*reinterpret_cast<const uintx4*>(a + (i / 2) * (32 * 64) + ao[i % 2] + pl * kXhPlane));
    };
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
      for (int pl = 0; pl < NP; ++pl) y[c2][pl] = as_bf16x8(*reinterpret_cast<const uintx4*>(b + (c2 * 3 + pl) * 1024));
    read(0);
    between();
    if (FWD && s > 0) { c[KT - 1] += late; asm volatile("" : "+v"(c[KT - 1])); }
    floatx16 sum[2];
    // (the next step's operands are requested before this one's products; fences keep the compiler from holding more of them)
#pragma unroll
    for (int i = 0; i < 2 * KT; ++i) {
      const int t = i / 2, c2 = i % 2;
      if (i + 1 < 2 * KT) read(i + 1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (FWD) {
        // (added to the tile's sum once the next tile's products are on their way)
        floatx16& l = sum[t % 2];
        if (c2 == 0) {
#pragma unroll
          for (int v = 0; v < 16; ++v) l[v] = 0.f;
        }
        // (smallest terms first)
        l = CAFEQ_MFMA_BF16(x[c2][2], y[c2][0], l);
        if constexpr (NP == 3) {
          l = CAFEQ_MFMA_BF16(x[c2][0], y[c2][2], l);
          l = CAFEQ_MFMA_BF16(x[c2][1], y[c2][1], l);
        }
        l = CAFEQ_MFMA_BF16(x[c2][1], y[c2][0], l);
        if constexpr (NP == 3) l = CAFEQ_MFMA_BF16(x[c2][0], y[c2][1], l);
        l = CAFEQ_MFMA_BF16(x[c2][0], y[c2][0], l);
        if (c2 == 0 && t > 0) {
          c[t - 1] += sum[(t + 1) % 2];
          asm volatile("" : "+v"(c[t - 1]));               // (now, and not at the end of the loop)
        }
      } else {
        c[t] = CAFEQ_MFMA_BF16(x[c2][1], y[c2][0], c[t]);
        c[t] = CAFEQ_MFMA_BF16(x[c2][0], y[c2][1], c[t]);
        c[t] = CAFEQ_MFMA_BF16(x[c2][0], y[c2][0], c[t]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (FWD) late = sum[(KT - 1) % 2];
  };
  const std::integral_constant<bool, true> ahead{};
  const std::integral_constant<bool, false> backward{};
  const std::integral_constant<int, WP> wparts{};
  const std::integral_constant<int, 2> eparts{};

  dma(p.Afwd, kXhFwd, cb, 0, fwd_at(0));
  load_w(seg, mis, 0, 16);

  // running sums per lane
  float s_l2 = 0.f, s_errz = 0.f, s_wsq = 0.f, s_sur = 0.f, s_va2[NG], m_ref = -INFINITY;
#pragma unroll
  for (int i = 0; i < NG; ++i) s_va2[i] = 0.f;
  const bool lse = INV && p.loss_kind == kLossLse;
  auto flush = [&](int sg) {
    float vals[kHdrVa2 + NGS];
    vals[kHdrL2] = s_l2; vals[kHdrErrZ] = s_errz; vals[kHdrWsq] = s_wsq; vals[kHdrSur] = s_sur;
    vals[kHdrMref] = 0.f; vals[5] = 0.f; vals[6] = 0.f; vals[7] = 0.f;
#pragma unroll
    for (int i = 0; i < NGS; ++i) vals[kHdrVa2 + i] = (NGS == 1 ? half == 0 : i / NG == half) ? s_va2[i % NG] : 0.f;
#pragma unroll
    for (int i = 0; i < kHdrVa2 + NGS; ++i) {
      const float t = wave_sum(vals[i]);
      if (lane == 0) hred[wave * kHdrFloats + i] = t;
    }
    __syncthreads();
    if (tid < kHdrVa2 + NGS) {
      float t = 0.f;
#pragma unroll
      for (int ww = 0; ww < kXhWaves; ++ww) t += hred[ww * kHdrFloats + tid];
      if (tid == kHdrMref) t = m_ref;
      p.slot_hdr[(w + sg) * kHdrFloats + tid] = t;
    }
    __syncthreads();
    s_l2 = s_errz = s_wsq = s_sur = 0.f;
#pragma unroll
    for (int i = 0; i < NG; ++i) s_va2[i] = 0.f;
    m_ref = -INFINITY;
  };

  for (int64_t mt = mt0; mt < mt1; ++mt) {
    if (seg != cur_seg) {
      if constexpr (INV) flush(cur_seg);
      cur_seg = seg;
    }
    const int64_t line = int64_t(mis) * kMacroLines + strip * kStripLines + ln;
    const bool valid = line < p.nlines;
    const int64_t ax0 = int64_t(seg) * K + 128 * half;
    int nseg_ = seg, nmis = mis + 1;
    if (nmis == mt_per_seg) { nmis = 0; ++nseg_; }
    // (the last macro-tile requests itself once more: every step issues the same requests)
    const bool has_next = mt + 1 < mt1;
    const int pseg = has_next ? nseg_ : seg, pmis = has_next ? nmis : mis, nbk = blk_id(pseg);

    if (!valid) {
#pragma unroll
      for (int f = 0; f < 64; ++f) wreg[f] = 0.f;
    }
    if constexpr (INV) {
#pragma unroll
      for (int f = 0; f < 64; ++f) s_wsq = fmaf(wreg[f], wreg[f], s_wsq);
    }
    asm volatile("" : "+v"(s_wsq));                  // (sums are taken where they stand, not where registers are short)
    if (half == 0) put(wparts, wreg, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // stage 0 has landed
    __syncthreads();

    // ---- forward transform
    floatx16 acc[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    floatx16 late;
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      if (s + 1 < NST) dma(p.Afwd, kXhFwd, cb, s + 1, fwd_at(s + 1));
      else if (INV) dma(p.Ainv, kXhBack, cb, 0, back_at(0));
      else dma(p.Afwd, kXhFwd, nbk, 0, fwd_at(0));
      products(ahead, acc, late, fwd_at(s), s, [&]() __attribute__((always_inline)) {
        if (s + 1 < NST && half == (s + 1) / 4) put(wparts, wreg + 16 * ((s + 1) % 4), s + 1);
      });
      vm_wait(0);                                    // the next stage has landed
      __syncthreads();
    }
    if constexpr (INV) dma(p.Ainv, kXhBack, cb, 1, back_at(1));
    acc[KT - 1] += late;
    if constexpr (MODE == kXhCorrect) {
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] += wreg[16 * t + v];
    }
    if constexpr (!INV) load_w(pseg, pmis, 0, 16);

    if constexpr (MODE == kXhApply) {
      if (valid) {
        if (AXIS == CAFEQ_AXIS_COL) {
          float* dst = p.Zout + line * p.cols + ax0 + 4 * h;
#pragma unroll
          for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              *reinterpret_cast<float4*>(dst + 32 * t + 8 * q) =
                  make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
        } else {
          const uint32_t loff = uint32_t(4 * h) * uint32_t(p.cols) + uint32_t(line);
#pragma unroll
          for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) (p.Zout + (ax0 + 32 * t + 8 * (v / 4) + (v % 4)) * p.cols)[loff] = acc[t][v];
        }
      }
    }

    if constexpr (MODE != kXhApply) {
      // ---- per group: absmax and arg-max; what the halves need of each other
      float tz[KT];                                  // per tile: signed value at the arg-max,
      int tj[KT];                                    // its index in the tile without the lane half's term
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        tz[t] = fabsf(acc[t][0]) > 0.f ? acc[t][0] : 0.f;
        tj[t] = 0;
      }
      auto step = [&](auto rc) __attribute__((always_inline)) {
        constexpr int R = decltype(rc)::value;
        argmax4<8 * (R / 4) + R % 4>(tz, tj, acc[0][R], acc[1][R], acc[2][R], acc[3][R]);
      };
      StaticFor<1, 16>::run(step);
      float gz[NG], zl = 0.f;                        // zl: the line's largest
      int gj[NG];
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        float zs = tz[gi * TPG];
        int j = 32 * gi * TPG + tj[gi * TPG];
#pragma unroll
        for (int t = gi * TPG + 1; t < (gi + 1) * TPG; ++t)
          if (fabsf(tz[t]) > fabsf(zs)) { zs = tz[t]; j = 32 * t + tj[t]; }
        j += 4 * h;
        const float oz = __shfl_xor(zs, 32);
        const int oj = __shfl_xor(j, 32);
        if (fabsf(oz) > fabsf(zs) || (fabsf(oz) == fabsf(zs) && oj < j)) { zs = oz; j = oj; }
        gz[gi] = zs;
        gj[gi] = G == 256 ? j + 128 * half : j - gi * G;      // index inside the group
        zl = fmaxf(zl, fabsf(zs));
      }
      if (G == 256 || lse) {
        if constexpr (G == 256)
          if (h == 0) { zsg[mine] = gz[0]; zix[mine] = gj[0]; }
        if (lse) {
          const float wm = cluster_allmax<64>(valid ? zl : 0.f);
          if (lane == 0) wvm[wave] = wm;
        }
        __syncthreads();
        if constexpr (G == 256) {
          const float oz = zsg[other];
          const int oj = zix[other];
          if (fabsf(oz) > fabsf(gz[0]) || (fabsf(oz) == fabsf(gz[0]) && oj < gj[0])) { gz[0] = oz; gj[0] = oj; }
        }
        if (lse) {
          // exponentials relative to a workgroup-wide running reference
          float nm = wvm[0];
#pragma unroll
          for (int ww = 1; ww < kXhWaves; ++ww) nm = fmaxf(nm, wvm[ww]);
          if (nm > m_ref) {
            s_sur *= __expf(p.lse_t * (m_ref - nm));          // 0 on the first macro-tile
            m_ref = nm;
          }
        }
      }
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        const int gs = G == 256 ? 0 : half * NG + gi;         // the group's number in the segment
        const bool own = h == 0 && (G != 256 || half == 0);   // who answers for the group
        const float zs = gz[gi], a = fabsf(zs);
        if (INV && p.rec && valid && own)
          p.rec[(int64_t(seg) * NGS + gs) * p.nlines + line] = make_float2(zs, __int_as_float(gj[gi]));
        const float inv = grid_inv(a, p.grid.qmax), s = grid_scale(a, p.grid.qmax);
        if (p.scales && valid && own) {
          const int64_t gidx = int64_t(seg) * NGS + gs;
          p.scales[AXIS == CAFEQ_AXIS_COL ? line * (p.cols / G) + gidx : gidx * p.cols + line] = s;
        }
#pragma unroll
        for (int f4 = gi * TPG * 4; f4 < (gi + 1) * TPG * 4; ++f4) {
          float q[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int f = 4 * f4 + e;
            const float z = acc[f / 16][f % 16];
            q[e] = grid_code(z, inv, p.grid);
            if constexpr (INV) {
              const float er = __fmul_rn(q[e], s) - z;
              s_errz = fmaf(er, er, s_errz);
              acc[f / 16][f % 16] = er;
            }
          }
          if (p.codes && valid) {
            const uint32_t pk = pack4(q[0], q[1], q[2], q[3]);
            const int j0 = 8 * f4 + 4 * h;
            if (AXIS == CAFEQ_AXIS_COL) {
              *reinterpret_cast<uint32_t*>(p.codes + line * p.cols + ax0 + j0) = pk;
            } else {
              int8_t* rowp = p.codes + (ax0 + 8 * f4) * p.cols;
              const uint32_t loff = uint32_t(4 * h) * uint32_t(p.cols) + uint32_t(line);
#pragma unroll
              for (int e = 0; e < 4; ++e) rowp[loff + uint32_t(e) * uint32_t(p.cols)] = int8_t(pk >> (8 * e));
            }
          }
        }
        if constexpr (INV) {
          const float a2 = a * a;
          if (own) {
            s_va2[gi] += a2;
            if (!lse) s_sur = fmaf(a2, p.rG[seg * NGS + gs], s_sur);
            else if (valid) s_sur += __expf(p.lse_t * (a - m_ref));
          }
        }
      }

      // ---- inverse transform of the errors and the l2 proxy
      if constexpr (INV) {
        float err[64];
#pragma unroll
        for (int f = 0; f < 64; ++f) err[f] = acc[f / 16][f % 16];
        asm volatile("" : "+v"(s_errz));
        if (half == 0) put(eparts, err, 0);
        __syncthreads();
        floatx16 d[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
          for (int v = 0; v < 16; ++v) d[t][v] = 0.f;
#pragma unroll
        for (int s = 0; s < NST; ++s) {
          if (s + 2 < NST) dma(p.Ainv, kXhBack, cb, s + 2, back_at(s + 2));
          else if (s + 1 == NST) dma(p.Afwd, kXhFwd, nbk, 0, fwd_at(0));
          // the next strip's weights, where the errors leave their registers, behind the step's fill
          if (s >= 4) load_w(pseg, pmis, 4 * (s - 4), 4 * (s - 3));
          products(backward, d, d[0], back_at(s), s, [&]() __attribute__((always_inline)) {
            if (s + 1 < NST && half == (s + 1) / 4) put(eparts, err + 16 * ((s + 1) % 4), s + 1);
          });
          // younger than the next stage's fill: this step's, and this step's and the last one's weights
          if (s + 1 < NST) vm_wait((s + 2 < NST ? NFB : 0) + (s >= 4 ? 4 * NWL : 0) + (s >= 5 ? 4 * NWL : 0));
          __syncthreads();
        }
        float l2 = 0.f;
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
          for (int v = 0; v < 16; ++v) l2 = fmaf(d[t][v], d[t][v], l2);
        s_l2 += l2;
      }
    }
    seg = nseg_;
    mis = nmis;
    cb = nbk;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the last macro-tile's requests for a next one)
  if constexpr (INV) flush(cur_seg);
}

template <int G, int AXIS, XhMode MODE, bool B16>
int launch_x256_t(const CoreParams& p, hipStream_t st) {
  const auto kern = xform256_kernel<G, AXIS, MODE, B16>;
  static std::atomic<bool> attr_set{false};   // per instantiation
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kXhLds) != hipSuccess)
      return CAFEQ_ERR_LAUNCH;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3(unsigned(p.nwg)), dim3(kXhThreads), kXhLds, st, p);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
template <int G, int AXIS, XhMode MODE>
int launch_x256(const CoreParams& p, hipStream_t st) {
  if constexpr (MODE == kXhCorrect) {
    return p.dtype == CAFEQ_F32 ? launch_x256_t<G, AXIS, MODE, false>(p, st) : int(CAFEQ_ERR_UNSUPPORTED);
  } else {
    return p.dtype == CAFEQ_F32 ? launch_x256_t<G, AXIS, MODE, false>(p, st) : launch_x256_t<G, AXIS, MODE, true>(p, st);
  }
}
template <int G>
int launch_x256(int axis, const CoreParams& p, hipStream_t st) {
  const bool col = axis == CAFEQ_AXIS_COL;
  if (p.do_inverse) return col ? launch_x256<G, CAFEQ_AXIS_COL, kXhLoss>(p, st) : launch_x256<G, CAFEQ_AXIS_ROW, kXhLoss>(p, st);
  return col ? launch_x256<G, CAFEQ_AXIS_COL, kXhCorrect>(p, st) : launch_x256<G, CAFEQ_AXIS_ROW, kXhCorrect>(p, st);
}

}  // namespace

int launch_xform256(int G, int axis, const CoreParams& p, hipStream_t st) {
  if (p.fscale || !p.Afwd || p.do_grad || (p.do_inverse && !p.Ainv)) return CAFEQ_ERR_INVALID_ARG;
  if (p.Zout)
    return axis == CAFEQ_AXIS_COL ? launch_x256<256, CAFEQ_AXIS_COL, kXhApply>(p, st) : launch_x256<256, CAFEQ_AXIS_ROW, kXhApply>(p, st);
  switch (G) {
    case 32: return launch_x256<32>(axis, p, st);
    case 64: return launch_x256<64>(axis, p, st);
    case 128: return launch_x256<128>(axis, p, st);
    case 256: return launch_x256<256>(axis, p, st);
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
}

}  // namespace cafeq
