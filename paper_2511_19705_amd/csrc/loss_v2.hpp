// Loss pass over PREPARED weights for transform blocks of 32, 64 and 128 (paper Sec. 4 / 4.1 / 4.2: transform,
// per-group absmax quantizer, inverse transform of the rounding error, l2 proxy, surrogate partials).  A segment of 128 holds
// 128 / K blocks.  Blocks of 64 and 32 this way, and before that in the general kernel with six bfloat16 products and the
// gradient on its way: 2B-shaped matrix at k = 64 34.7 us (76; without the gradient 47); whole evaluations of 2304 x 9216
// pairs with groups of 128 92 us (176) at k = 64, 84 (161) at k = 32.
//
// The weights are constant over the tens of thousands of evaluations of a learning run, so
// cafeq_prepare_weights() stores them once in the form the matrix cores consume: per tile of 32 lines x
// 128 axis indices, two float16 parts (hi + lo of the line scaled by a power of two to [2^3, 2^4)) laid
// out so that one 16-byte load per lane is the B operand of one MFMA step -- the same 4 bytes per element
// as float32, no per-call splitting, every load a contiguous kilobyte per wave.  ||W||^2 and the per-line
// scale factors are stored beside them.
//
// Kernel shape.  One workgroup of eight waves per compute unit (two waves per SIMD).  The operand planes of
// the current block -- T and T^-1, float16 hi and lo parts each, 128 KB -- stay in LDS for as long as
// the workgroup works inside one segment, so they are fetched once per segment instead of once per
// macro-tile.  Each wave owns strips of 32 lines and alternates between a matrix phase
//   M(i) = inverse transform of strip i-1's error  +  forward transform of strip i
// and a vector phase
//   V(i) = quantizer epilogue of strip i (scale back, group absmax / arg-max, codes, error, records)
// with one workgroup barrier per phase; waves 4-7 run one phase behind waves 0-3, so that on every SIMD one
// wave feeds the matrix pipe while the other occupies the vector pipe (two independent workgroups drift
// into running the same phase at the same time and then share each pipe in turn).
//
// Arithmetic.  Forward: three float16 part products (hi.hi, hi.lo, lo.hi), float32 accumulation, exact
// scaling back by powers of two.  The scalings -- a line's weights below 2^4, a block's entries below 2^5 --
// bound every accumulator by 128 * 2^9 = 2^16, so the rounding error of the quantizer, at most half a step
// = absmax / (2 qmax) <= 2^15 in accumulator units, is a float16 number without any rescaling (the matrix
// cores take denormal float16 inputs exactly, so small entries lose nothing).  Inverse: the error E as ONE
// float16 part (round to nearest even: 2^-12 relative, zero mean) times T^-1 as hi + lo (2^-22 relative: a
// fixed operand's rounding would otherwise bias every element the same way).  Blocks of 32 and 64 take the error in two parts,
// blocks of 32 the forward operand in three (v2_fwd_parts), and a block that is far smaller than its line's others a scale of its
// own (rescale_strip: Student-t weights with outliers, 2304 x 9216 at k = 64, evaluation 75.5 -> 80.3 us for it, Gaussian ones nothing).
#pragma once
#include <atomic>

#include "gj_panel.hpp"   // StaticFor
#include "xform_core.hpp"

namespace cafeq {

namespace {

constexpr int kV2Waves = 8;
constexpr int kV2Threads = kV2Waves * 64;
constexpr int kV2MacroLines = kV2Waves * 32;
// one prepared tile: [8 steps][parts][64 lanes][16 B].  Two parts for float32 weights, one for bfloat16: eight significant
// bits are a float16 number (what lies below 2^-24 of a line scaled to 2^4 is below the second part's reach as well), so
// the second part was zeros: half the bytes, four products a strip and step instead of five, the same results bit for bit
// (27B-shaped pair, with argmax4 below: loss pass 370 -> 334 us, gradient pass 328 -> 246 us; codes of its gate
// 223 -> 174 us).
constexpr int v2_tile_bytes(int parts) { return 32 * 128 * 2 * parts; }
// operand planes of a segment (T and T^-1, 64 KB each for blocks of 128), the waves' sums
constexpr int v2_lds(int K) { return (2 * v2_fwd_parts(K) + 4) * 128 * K + kV2Waves * kHdrFloats * 4 + 64 + kV2Waves * 2 * 8; }

// Marks in a line's scale, a power of two: 32 (64) of its inputs are far smaller than the segment's largest
constexpr uint32_t kFar32 = 1, kFar64 = 2;
// A scaled weight as float16 parts.  (One part: the second is zero, or not a number behind an infinity, which then is none
// either, as in two parts.)
__device__ __forceinline__ void weight_parts(float y, bool one, uint32_t* hi, uint32_t* lo) {
  const _Float16 p0 = _Float16(y);
  const _Float16 p1 = _Float16(y - float(p0));
  *hi = __builtin_bit_cast(uint16_t, one && !(p1 == _Float16(0)) ? p1 : p0);
  *lo = __builtin_bit_cast(uint16_t, p1);
}

// bidx: the workgroup's index among the p.nwg workgroups that share the matrix; WP: parts of the prepared weights;
// REC: write the arg-max records (the gradient pass follows); OUT: write scales and / or codes
// SELF (blocks of 64 and 128): the operand planes are split here, from T and T^-1 themselves -- the same bytes to read as the planes, once
// per workgroup and segment -- instead of by a launch of their own, and the groups' sums of rho are taken on the way;
// PAIR: a member of a pair (kLossLse)
template <int K, int G, int AXIS, bool REC, bool OUT, int WP, bool SELF, bool PAIR>
__device__ __forceinline__ void loss_v2_body(const CoreParams& p, const unsigned bidx) {
  constexpr int L = 128, KT = 4, NGRP = L / G, RPG = G / 2;
  // blocks per segment, output tiles and steps of 16 inputs of a block
  constexpr int NB = L / K, BT = K / 32, CB = K / 16;
  // float16 parts of the forward operand and of the error, bytes of a block's planes and of a segment's
  constexpr int FP = v2_fwd_parts(K), EP = v2_err_parts(K);
  constexpr int FBLKB = 2 * FP * K * K, IBLKB = 4 * K * K, FPLB = NB * FBLKB, IPLB = NB * IBLKB;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* lfw = smem;                      // forward planes [block][K / 32 stages][part][K rows][64 B]
  unsigned char* liv = smem + FPLB;               // inverse planes, likewise
  float* hred = reinterpret_cast<float*>(smem + FPLB + IPLB);   // [8 waves][kHdrFloats]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2;                      // phase group: waves 4-7 run one phase behind (waves i and i + 4 share a SIMD)
  const int ln = lane & 31, h = lane >> 5;

  int64_t w = bidx;
  if ((p.nwg & 7) == 0) w = int64_t(bidx & 7) * (p.nwg >> 3) + (bidx >> 3);
  const int64_t mt0 = chunk_begin(w, p.n_mt, p.nwg), mt1 = chunk_begin(w + 1, p.n_mt, p.nwg);
  if (mt0 >= mt1) return;
  const int mt_per_seg = int(p.mt_per_seg);       // macro-tiles of 256 lines per segment
  const int64_t nlp = int64_t(mt_per_seg) * kV2MacroLines;
  const bool lse_on = PAIR || p.loss_kind == kLossLse;
  const int swz = (ln >> 2) & 3;
  const int aoff0 = ln * 64 + ((h ^ swz) << 4), aoff1 = ln * 64 + (((2 + h) ^ swz) << 4);
  bool wsq_pending = w == 0;

  // per-lane running sums of the current segment
  float s_l2 = 0.f, s_errz = 0.f, s_sur = 0.f, m_ref = -INFINITY;
  float s_va2[NGRP];
#pragma unroll
  for (int i = 0; i < NGRP; ++i) s_va2[i] = 0.f;

  // Prepared B operands of the strip the next forward phase transforms, and that strip's line scale factor.
  // They are requested a whole vector phase ahead of their use (at the start of the vector phase of the strip
  // before, across run boundaries too), so that their latency never reaches the matrix pipe: requested at the
  // start of the matrix phase they had only the inverse transform (about a microsecond) to arrive in.
  uintx4 wq[8 * WP];
  float lsc_nx = 0.f;
  // (NB > 1) a line's blocks against the line's scale: a byte of binary exponent each, zero but in strips that rescale_strip took
  int xe = 0;
  auto xe_of = [&](int b) { return int(uint32_t(xe) << (24 - 8 * b)) >> 24; };
  auto request_strip = [&](int sg, int64_t strip) {   // strip: the wave's strip inside segment sg
    lsc_nx = p.prep_lscale[int64_t(sg) * nlp + strip * 32 + ln];
    const unsigned char* tp = p.prep_planes + (int64_t(sg) * (nlp / 32) + strip) * v2_tile_bytes(WP) + lane * 16;
#pragma unroll
    for (int i = 0; i < 8 * WP; ++i) wq[i] = *reinterpret_cast<const uintx4*>(tp + i * 1024);
  };
  // Blocks of 32 and 64 share their line's scale with the segment's other blocks.  One that is far smaller would keep few of
  // its bits (a thousand times: maxima to 5e-7, against 6e-8).  Such lines are marked in their scale; a strip that holds one --
  // one in a hundred at k = 64, one in twenty at k = 32 where weights are Student-t with outliers of twenty times -- is split anew
  // from the weights themselves, every block with a scale of its own.
  auto rescale_strip = [&](int sg, int64_t strip) {
    if constexpr (NB > 1) {
      xe = 0;
      if (!__any((__float_as_uint(lsc_nx) & (K == 32 ? kFar32 : kFar64)) != 0)) return;
      // (nothing of this is worth a register in the other strips: kept apart from what could be worked out ahead)
      int own = lane;
      int64_t ld = p.ld, nl = p.nlines;
      const void* src = AXIS == CAFEQ_AXIS_COL ? p.W : p.prep_lines;
      asm volatile("" : "+v"(own), "+s"(ld), "+s"(nl), "+s"(src));
      const int64_t line = strip * 32 + (own & 31);
      const bool in = line < nl;
      const int64_t at = (AXIS == CAFEQ_AXIS_COL ? (in ? line : 0) * ld + int64_t(sg) * L : (int64_t(sg) * nlp + line) * L) + 8 * (own >> 5);
      // the weights as they are, where their parts will be: a step's eight inputs
#pragma unroll
      for (int i = 0; i < 8 * WP; ++i)
        wq[i] = *reinterpret_cast<const uintx4*>(static_cast<const unsigned char*>(src) + (at + 16 * (i / WP)) * (2 * WP) + 16 * (i % WP));
      auto input = [&](int cw, int e) {
        const uint32_t u = WP == 2 ? wq[2 * cw + e / 4][e % 4] : (e & 1 ? wq[cw][e / 2] & 0xFFFF0000u : wq[cw][e / 2] << 16);
        return in ? __uint_as_float(u) : 0.f;
      };
      const int exl = int(__float_as_uint(lsc_nx) >> 23 & 255u) + 3;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        float mx = 0.f;
#pragma unroll
        for (int i = 0; i < 8 * CB; ++i) {
          const float x = fabsf(input(CB * b + i / 8, i % 8));
          if (x < INFINITY) mx = fmaxf(mx, x);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        int ex = int(__float_as_uint(mx) >> 23);
        ex = ex < 4 ? 4 : (ex > 254 ? 254 : ex);
        // (a group's step in the units of its smallest block stays a number)
        if (ex < exl - (G > K ? 60 : 127)) ex = exl - (G > K ? 60 : 127);
        xe |= ((ex - exl) & 255) << (8 * b);
        const float wsc = __uint_as_float(uint32_t(257 - ex) << 23);
#pragma unroll
        for (int cw = CB * b; cw < CB * (b + 1); ++cw) {
          uint32_t hi[8], lo[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) weight_parts(input(cw, e) * wsc, WP == 1, &hi[e], &lo[e]);
#pragma unroll
          for (int e2 = 0; e2 < 4; ++e2) {
            wq[WP * cw][e2] = hi[2 * e2] | (hi[2 * e2 + 1] << 16);
            if constexpr (WP == 2) wq[2 * cw + 1][e2] = lo[2 * e2] | (lo[2 * e2 + 1] << 16);
          }
        }
      }
    }
  };
  // (The variants that write codes or scales from two-part weights keep their requests at the start of the matrix phase:
  // their vector phase has no registers to hold a strip in flight.  One part fits: codes of the 27B-shaped gate in
  // bfloat16 185 -> 173 us.)
  constexpr bool EARLY = !OUT || WP == 1;
  // (16-byte code stores need the code matrix aligned to 16 bytes; its row length is a multiple of 128)
  const bool wide_codes = OUT && (reinterpret_cast<uintptr_t>(p.codes) & 15) == 0;
  if constexpr (EARLY) {
    const int sg = int(mt0 / mt_per_seg);
    request_strip(sg, (mt0 - int64_t(sg) * mt_per_seg) * kV2Waves + wave);
  }

  // (SELF) the segment's planes into LDS, as split_planes_kernel (aux_kernels.hip) writes them: a block scaled by the power of two that
  // puts its largest finite magnitude into [2^4, 2^5), two float16 parts; the factors back.  A thread takes one 16-byte vector of
  // each of a block's stages (K = 64: of one of the two).  With want_rg (single matrices: blocks of 64) also the sums of T^-1's
  // squares over each group's indices, the contraction's: into rg, and to memory for the gradient pass (workgroups that share a segment write
  // the same).
  double* rsum = reinterpret_cast<double*>(hred + kV2Waves * kHdrFloats + 16);   // [8 waves][2]
  auto split_blocks = [&](const int (&bid)[NB], float (&fwd_back)[NB], float (&inv_back)[NB], bool want_rg, int sg, float (&rg)[NGRP])
      __attribute__((always_inline)) {
    constexpr bool TR = AXIS == CAFEQ_AXIS_COL;    // the operands' rows are the blocks' columns
    static_assert(!SELF || ((PAIR && K == 128 || K == 64) && FP == 2), "blocks of 64, pairs' blocks of 128");
    constexpr int NS = K == 128 ? 4 : 1, LK = K == 128 ? 7 : 6;
    // (transposed: lanes along a row of the block, a contraction index each; else four lanes along 128 bytes of a row)
    const int out = TR ? tid & (K - 1) : (tid >> 2) & (K - 1), cq = TR ? (tid >> LK) & 3 : tid & 3, c2 = cq >> 1, hh = cq & 1;
    const int st0 = K == 128 ? 0 : wave >> 2;
    float x[2][NB][NS][8];
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const float* src = (o ? p.Tback : p.Tfwd) + int64_t(bid[b]) * K * K;
#pragma unroll
        for (int st = 0; st < NS; ++st)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            // inputs in runs of four: forward eight side by side, back two runs eight apart (the accumulators' order)
            const int in = 32 * (st0 + st) + 16 * c2 + (o ? 8 * u + 4 * hh : 8 * hh + 4 * u);
            float (&y)[8] = x[o][b][st];
            if constexpr (TR) {
#pragma unroll
              for (int e = 0; e < 4; ++e) y[4 * u + e] = src[(in + e) * K + out];
            } else {
              const float4 v = *reinterpret_cast<const float4*>(src + out * K + in);
              y[4 * u] = v.x; y[4 * u + 1] = v.y; y[4 * u + 2] = v.z; y[4 * u + 3] = v.w;
            }
          }
      }
    if (want_rg) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        double t = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) t += double(x[1][b][0][e]) * x[1][b][0][e];
        t = wave_sum(t);
        if (lane == 0) rsum[wave * 2 + b] = t;
      }
    }
    float mx[2][NB];
    for (int finite = 0; finite < 2; ++finite) {   // (infinite entries are looked for only where there is one)
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          float m = 0.f;
#pragma unroll
          for (int st = 0; st < NS; ++st)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float a = fabsf(x[o][b][st][e]);
              m = fmaxf(m, finite && !(a < INFINITY) ? 0.f : a);
            }
          m = cluster_allmax<64>(m);
          if (lane == 0) hred[wave * kHdrFloats + o * NB + b] = m;
        }
      __syncthreads();
      bool all = true;
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          mx[o][b] = hred[o * NB + b];
#pragma unroll
          for (int ww = 1; ww < kV2Waves; ++ww) mx[o][b] = fmaxf(mx[o][b], hred[ww * kHdrFloats + o * NB + b]);
          all = all && mx[o][b] < INFINITY;
        }
      if (all) break;
      __syncthreads();
    }
    if (want_rg) {
#pragma unroll
      for (int gi = 0; gi < NGRP; ++gi) {
        double t = 0;
        for (int ww = 0; ww < kV2Waves; ++ww)
#pragma unroll
          for (int b = 0; b < NB; ++b)
            if ((b * K + 32 * (ww >> 2)) / G == gi) t += rsum[ww * 2 + b];
        rg[gi] = float(t);
        if (tid == 0) p.rG_out[int64_t(sg) * NGRP + gi] = rg[gi];
      }
    }
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        int ex = int(__float_as_uint(mx[o][b]) >> 23);
        ex = ex < 32 ? 32 : (ex > 254 ? 254 : ex);
        const float sc = __uint_as_float(uint32_t(258 - ex) << 23);
        (o ? inv_back[b] : fwd_back[b]) = __uint_as_float(uint32_t(ex - 4) << 23);
        unsigned char* at = (o ? liv + b * IBLKB : lfw + b * FBLKB) + st0 * (2 * K * 64) + out * 64 + ((cq ^ ((out >> 2) & 3)) << 4);
#pragma unroll
        for (int st = 0; st < NS; ++st) {
          uintx4 hi, lo;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float y0 = x[o][b][st][2 * i] * sc, y1 = x[o][b][st][2 * i + 1] * sc;
            const uint32_t both = pack_f16(y0, y1);
            const halfx2 hb = __builtin_bit_cast(halfx2, both);
            hi[i] = both;
            lo[i] = pack_f16(y0 - float(hb[0]), y1 - float(hb[1]));
          }
          *reinterpret_cast<uintx4*>(at + st * (2 * K * 64)) = hi;
          *reinterpret_cast<uintx4*>(at + st * (2 * K * 64) + K * 64) = lo;
        }
      }
  };

  for (int64_t mt = mt0; mt < mt1;) {
    const int seg = int(mt / mt_per_seg);
    const int mis0 = int(mt - int64_t(seg) * mt_per_seg);
    const int n = int(mt1 - mt < int64_t(mt_per_seg - mis0) ? mt1 - mt : int64_t(mt_per_seg - mis0));
    // ---- the segment's operand planes into LDS (the previous segment's readers are past flush's barriers)
    // Several blocks of a segment (K < 128) have a scale each.  A block's accumulators and errors stay in its own units --
    // rel[i] of the segment's, the largest -- and a group that spans blocks is measured in the segment's: the factors, powers
    // of two, are applied to its maxima and to the reciprocal and the step that each block's elements see.
    int bid[NB];
    float fsc = 0.f, fsf[NB], fsi[NB], rel[NB], inv_rel[NB], cl2[NB];
    float rgs[NGRP];          // (SELF) the segment's groups: sums of rho
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      bid[i] = p.rep != 1 ? (seg * NB + i) / p.rep : seg * NB + i;   // (rep is 1 on the column axis)
      if constexpr (!SELF) {
        fsf[i] = p.fscale[bid[i]];
        fsi[i] = p.fscale_inv[bid[i]];
      }
    }
    if constexpr (SELF) split_blocks(bid, fsf, fsi, !PAIR && !lse_on, seg, rgs);
#pragma unroll
    for (int i = 0; i < NB; ++i) fsc = fmaxf(fsc, fsf[i]);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      rel[i] = NB == 1 ? 1.f : fsf[i] / fsc;
      inv_rel[i] = NB == 1 ? 1.f : fsc / fsf[i];
      cl2[i] = (rel[i] * fsi[i]) * (rel[i] * fsi[i]);       // (NB > 1) squared transformed error: segment's units -> per line's
    }
    if constexpr (!SELF) {
      constexpr int NF = FPLB / (16 * kV2Threads), NI = IPLB / (16 * kV2Threads);   // vectors per thread
      static_assert(FPLB % (16 * kV2Threads) == 0 && IPLB % (16 * kV2Threads) == 0, "whole vectors");
      uintx4 tf[NF], ti[NI];
      auto fetch = [&](const uint16_t* base, int v, int blkb) {
        const int blk = v / (blkb / 16);
        int bb = bid[0];
#pragma unroll
        for (int q = 1; q < NB; ++q) bb = blk == q ? bid[q] : bb;
        return *reinterpret_cast<const uintx4*>(reinterpret_cast<const unsigned char*>(base) + int64_t(bb) * blkb +
                                                int64_t(v % (blkb / 16)) * 16);
      };
#pragma unroll
      for (int i = 0; i < NF; ++i) tf[i] = fetch(p.Afwd, i * kV2Threads + tid, FBLKB);
#pragma unroll
      for (int i = 0; i < NI; ++i) ti[i] = fetch(p.Ainv, i * kV2Threads + tid, IBLKB);
#pragma unroll
      for (int i = 0; i < NF; ++i) reinterpret_cast<uintx4*>(lfw)[i * kV2Threads + tid] = tf[i];
#pragma unroll
      for (int i = 0; i < NI; ++i) reinterpret_cast<uintx4*>(liv)[i * kV2Threads + tid] = ti[i];
    }
    __syncthreads();

    float usc = 0.f;          // the factor back to the units of Z for the strip in the accumulators
    float usc2_prev = 0.f;    // its square for the strip whose error the next inverse phase transforms
    floatx16 acc[KT];
    uint32_t ebf[L / 4], elo[EP == 2 ? L / 4 : 1];   // the error as packed float16 (accumulator units): B operands of the inverse phase
    // the strip after strip m of this run: the run's next one, else the first of the next run (the next segment),
    // else -- the range ends here -- strip m once more (an unconditional request keeps the wait counts exact)
    const bool more_runs = mt + n < mt1;
    auto request_next = [&](int m) {
      int sg = seg;
      int64_t strip = int64_t(mis0 + m + 1) * kV2Waves + wave;
      if (m + 1 == n) {
        if (more_runs) { sg = seg + 1; strip = wave; }
        else strip -= kV2Waves;
      }
      request_strip(sg, strip);
    };

    // Both contractions walk the output tiles one after the other (tile t: 32 outputs, its accumulator a
    // chain of MFMAs over the eight steps of 16 inputs), so that only a few operand registers are live: the
    // A operands (transform tiles from LDS) are requested two steps ahead into a rotating set of three, the
    // B operands are the lane's own registers.  Scheduling barriers pin the issue order per step: the LDS reads
    // of step + 2, then the step's MFMAs and vector work (the compiler would otherwise sink each read to just
    // before its use and wait for it there).
    //
    // matrix phase, second half: forward transform of the strip in wq
    auto forward = [&]() {
      const unsigned char* b0 = lfw + aoff0;
      const unsigned char* b1 = lfw + aoff1;
      auto frag = [&](int i, int pl) {   // i = CB t + c
        const int t = i / CB, c = i % CB;
        return *reinterpret_cast<const uintx4*>(((c & 1) ? b1 : b0) + (t / BT) * FBLKB + (c >> 1) * (FP * K * 64) + pl * (K * 64) + (t % BT) * (32 * 64));
      };
      // (three products a step cover two steps of LDS latency, two products four)
      constexpr int DF = WP == 2 ? 2 : 4;
      uintx4 fh[DF + 1], fl[DF + 1], fr[FP == 3 ? DF + 1 : 1];
      auto read = [&](int i) {
        fh[i % (DF + 1)] = frag(i, 0);
        fl[i % (DF + 1)] = frag(i, 1);
        if constexpr (FP == 3) fr[i % (DF + 1)] = frag(i, 2);
      };
#pragma unroll
      for (int i = 0; i < DF; ++i) read(i);
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        floatx16 a;
#pragma unroll
        for (int v = 0; v < 16; ++v) a[v] = 0.f;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
          const int i = CB * t + c, cw = (t / BT) * CB + c;   // cw: step of the segment
          if (i + DF < CB * KT) read(i + DF);
          __builtin_amdgcn_sched_barrier(0);     // the reads of step + DF are issued before this step's products
          const halfx8 xh = as_halfx8(fh[i % (DF + 1)]), xl = as_halfx8(fl[i % (DF + 1)]);
          const halfx8 vbh = as_halfx8(wq[WP * cw]);
          if constexpr (FP == 3) {
            a = CAFEQ_MFMA_F16(as_halfx8(fr[i % (DF + 1)]), vbh, a);
            if constexpr (WP == 2) a = CAFEQ_MFMA_F16(xl, as_halfx8(wq[WP * cw + 1]), a);
          }
          a = CAFEQ_MFMA_F16(xl, vbh, a);
          if constexpr (WP == 2) a = CAFEQ_MFMA_F16(xh, as_halfx8(wq[WP * cw + 1]), a);
          a = CAFEQ_MFMA_F16(xh, vbh, a);
          __builtin_amdgcn_sched_barrier(0);
        }
        acc[t] = a;
      }
    };
    // matrix phase, first half: D^T = Ainv . E^T for the strip whose error is in ebf, and the sum of its squares
    // (a tile's sum runs in the shadow of the next tile's products)
    auto inverse = [&](float usc2_strip) {
      float l2 = 0.f, l2s = 0.f;    // in the units of the strip's accumulators
      const unsigned char* b0 = liv + aoff0;
      const unsigned char* b1 = liv + aoff1;
      auto frag = [&](int i, int pl) {
        const int t = i / CB, c = i % CB;
        return *reinterpret_cast<const uintx4*>(((c & 1) ? b1 : b0) + (t / BT) * IBLKB + (c >> 1) * (2 * K * 64) + pl * (K * 64) + (t % BT) * (32 * 64));
      };
      // (two products per step cover only 64 cycles of matrix time, so the reads run four steps ahead)
      constexpr int DI = 4;
      uintx4 fh[DI + 1], fm[DI + 1];
#pragma unroll
      for (int i = 0; i < DI; ++i) { fh[i] = frag(i, 0); fm[i] = frag(i, 1); }
      floatx16 dp;
#pragma unroll
      for (int v = 0; v < 16; ++v) dp[v] = 0.f;
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        floatx16 a;
#pragma unroll
        for (int v = 0; v < 16; ++v) a[v] = 0.f;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
          const int i = CB * t + c, cw = (t / BT) * CB + c;
          if (i + DI < CB * KT) { fh[(i + DI) % (DI + 1)] = frag(i + DI, 0); fm[(i + DI) % (DI + 1)] = frag(i + DI, 1); }
          __builtin_amdgcn_sched_barrier(0);
          const halfx8 xh = as_halfx8(fh[i % (DI + 1)]), xm = as_halfx8(fm[i % (DI + 1)]);
          const halfx8 ve = as_halfx8(ebf[4 * cw], ebf[4 * cw + 1], ebf[4 * cw + 2], ebf[4 * cw + 3]);
          a = CAFEQ_MFMA_F16(xm, ve, a);
          if constexpr (EP == 2) a = CAFEQ_MFMA_F16(xh, as_halfx8(elo[4 * cw], elo[4 * cw + 1], elo[4 * cw + 2], elo[4 * cw + 3]), a);
          a = CAFEQ_MFMA_F16(xh, ve, a);
#pragma unroll
          for (int v = 16 * c / CB; v < 16 * (c + 1) / CB; ++v) l2 = fmaf(dp[v], dp[v], l2);   // previous tile (zeros for the first)
          __builtin_amdgcn_sched_barrier(0);
        }
        dp = a;
        if constexpr (NB > 1) if (t > 0 && t % BT == 0) {   // the block before is complete
          l2s = fmaf(l2, ldexpf(cl2[t / BT - 1], 2 * xe_of(t / BT - 1)), l2s);
          l2 = 0.f;
        }
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) l2 = fmaf(dp[v], dp[v], l2);
      if constexpr (NB > 1) l2 = fmaf(l2, ldexpf(cl2[NB - 1], 2 * xe_of(NB - 1)), l2s);
      s_l2 = fmaf(l2, usc2_strip, s_l2);
    };
    // vector phase: the quantizer on strip m (accumulators -> error).  The accumulators hold Z / usc with usc a
    // power of two per line, and everything up to the error stays in those units: absmax, reciprocal, codes and
    // error scale exactly (q = rint(z' * fl(qmax / a')) is the recipe's rint(z * fl(qmax / a)) bit for bit), so
    // the 64 multiplications back to the units of Z are replaced by a few per group and per strip.  (The two
    // differ only where a group's absmax or scale would be a denormal float32, below 1e-37.)
    auto epilogue = [&](int m) {
      const int64_t line = int64_t(mis0 + m) * kV2MacroLines + wave * 32 + ln;
      const bool valid = line < p.nlines;
      const int64_t ax0 = int64_t(seg) * L;
      const float usc2 = usc * usc;
      const float dsc = usc * fsi[0];  // (NB == 1) inverse-transformed error: accumulator units -> units of W
      float e2 = 0.f;               // sum of squared errors of this strip in accumulator units
      constexpr bool SPAN = G > K;  // groups of several blocks
      auto rx = [&](int b) { return ldexpf(rel[b], xe_of(b)); };   // (NB > 1) a block's units in those of segment and line
      // signed value at the arg-max of each tile of 32 and its index in the tile (without the lane-half term)
      float tz[KT];
      int tj[KT];
      if constexpr (REC) {
        // (the first step is the compiler's, which knows how long after a matrix instruction its results may be read)
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
      }
#pragma unroll
      for (int gi = 0; gi < NGRP; ++gi) {
        float zs = 0.f;
        int jf = 0;
        constexpr int TPG = G / 32;
        // the group's units: its block's, or the segment's
        const float usg = NB == 1 || SPAN ? usc : usc * rx(gi * TPG / BT);
        if constexpr (REC) {
          if constexpr (SPAN) {
#pragma unroll
            for (int t = gi * TPG; t < (gi + 1) * TPG; ++t) tz[t] *= rx(t / BT);
          }
          zs = tz[gi * TPG];
          jf = 32 * gi * TPG + tj[gi * TPG];
#pragma unroll
          for (int t = gi * TPG + 1; t < (gi + 1) * TPG; ++t)
            if (fabsf(tz[t]) > fabsf(zs)) { zs = tz[t]; jf = 32 * t + tj[t]; }
        } else {
          float a0 = 0.f;
#pragma unroll
          for (int f = gi * RPG; f < (gi + 1) * RPG; f += 2) {
            if (SPAN && f % (16 * BT) == 0 && f > gi * RPG) {      // the next block
              zs = fmaxf(zs, a0 * rx(f / (16 * BT) - 1));
              a0 = 0.f;
            }
            a0 = fmaxf(fmaxf(fabsf(acc[f / 16][f % 16]), fabsf(acc[(f + 1) / 16][(f + 1) % 16])), a0);
          }
          zs = SPAN ? fmaxf(zs, a0 * rx(((gi + 1) * TPG - 1) / BT)) : a0;
        }
        float as = fabsf(zs);       // absmax in the group's units
        {
          const float oz = __shfl_xor(zs, 32);
          const float oa = fabsf(oz);
          if constexpr (REC) {
            int j = jf + 4 * h;
            const int oj = __shfl_xor(j, 32);
            if (oa > as || (oa == as && oj < j)) { as = oa; zs = oz; j = oj; }
            if (valid && h == 0)
              p.rec[(int64_t(seg) * NGRP + gi) * p.nlines + line] = make_float2(zs * usg, __int_as_float(j - gi * G));
          } else {
            as = fmaxf(as, oa);
          }
        }
        const float a = as * usg;   // exact
        float inv = grid_inv(as, p.grid.qmax);
        float s = grid_scale(as, p.grid.qmax);
        const float inv0 = inv, s0 = s;
        float e2b = 0.f;
        if (OUT && p.scales && valid && h == 0) {
          const int64_t gidx = ax0 / G + gi;
          const float st = grid_scale(a, p.grid.qmax);
          if (AXIS == CAFEQ_AXIS_COL) p.scales[line * (p.cols / G) + gidx] = st;
          else p.scales[gidx * p.cols + line] = st;
        }
#pragma unroll
        for (int f2 = gi * RPG / 2; f2 < (gi + 1) * RPG / 2; ++f2) {
          if (SPAN && f2 % (8 * BT) == 0) {              // a block's first elements: the group's grid in its units
            inv = inv0 * rx(f2 / (8 * BT));
            s = s0 * ldexpf(inv_rel[f2 / (8 * BT)], -xe_of(f2 / (8 * BT)));
          }
          float er[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int f = 2 * f2 + e;
            const float z = acc[f / 16][f % 16];
            // |z * inv| <= qmax (1 + 2^-23), so the rounded value is already inside the grid: no clamp.
            // The error is taken with one rounding, q s - z (the recipe's fl(q s) - z differs by 2^-24 |q s|,
            // at most 2e-6 of the error's own size on grids of up to 4 bits).
            const float q = __builtin_rintf(__fmul_rn(z, inv));
            er[e] = fmaf(q, s, -z);
            // kept for the optional code output; a value that is not a number gets the grid's lowest code, as in the
            // general pass (blocks of 128 write 0 for it)
            if constexpr (OUT) acc[f / 16][f % 16] = NB == 1 ? q : fmaxf(q, p.grid.qmin);
          }
          ebf[f2] = pack_f16(er[0], er[1]);
          if constexpr (EP == 2) {
            const halfx2 eh = __builtin_bit_cast(halfx2, ebf[f2]);
            elo[f2] = pack_f16(er[0] - float(eh[0]), er[1] - float(eh[1]));
          }
          // the sum of squared errors from the packed pair (one dot-product instruction per pair; the float16
          // rounding of an error is 2^-12 relative and random in sign, far below the sum's budget)
          if constexpr (NB == 1) {
            e2 = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2, ebf[f2]), __builtin_bit_cast(halfx2, ebf[f2]), e2, false);
          } else {
            e2b = fmaf(er[0], er[0], fmaf(er[1], er[1], e2b));
            if (f2 % (8 * BT) == 8 * BT - 1 || f2 == (gi + 1) * RPG / 2 - 1) {
              e2 = fmaf(e2b, rx(f2 / (8 * BT)) * rx(f2 / (8 * BT)), e2);
              e2b = 0.f;
            }
          }
        }
        const float a2 = a * a;
        if (h == 0) s_va2[gi] += a2;
        if (!PAIR && !lse_on && h == 0) s_sur = fmaf(a2, SELF ? rgs[gi] : p.rG[seg * NGRP + gi], s_sur);
        if (lse_on) {
          // exponentials relative to this wave's running reference
          const float am = valid ? a : 0.f;
          const float nm = fmaxf(cluster_allmax<64>(am), m_ref);
          if (nm > m_ref) {
            s_sur *= __expf(p.lse_t * (m_ref - nm));   // 0 on the first group
            m_ref = nm;
          }
          if (valid && h == 0) s_sur += __expf(p.lse_t * (a - m_ref));
        }
      }
      s_errz = fmaf(e2, usc2, s_errz);
      if (OUT && AXIS == CAFEQ_AXIS_COL && L == 128 && p.codes && wide_codes) {
        // A line's 128 codes are spread over its two lanes in alternating 4-byte words (word f4 of lane half h:
        // codes 8 f4 + 4 h ..).  Swapping the upper lanes' word a with the lower lanes' word a + 8 leaves codes
        // 0..63 in the lower lane and 64..127 in the upper one: four 16-byte stores per lane instead of sixteen
        // 4-byte ones.
        uint32_t wd[16];
#pragma unroll
        for (int f4 = 0; f4 < 16; ++f4) {
          const int f = 4 * f4;
          wd[f4] = pack4(acc[f / 16][f % 16], acc[f / 16][f % 16 + 1], acc[f / 16][f % 16 + 2], acc[f / 16][f % 16 + 3]);
        }
#pragma unroll
        for (int a = 0; a < 8; ++a) {
          const auto r = __builtin_amdgcn_permlane32_swap(wd[a], wd[a + 8], false, false);
          wd[a] = r[0];
          wd[a + 8] = r[1];
        }
        if (valid) {
          int8_t* dst = p.codes + line * p.cols + ax0 + 64 * h;
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            uintx4 v;
            v[0] = wd[2 * m]; v[1] = wd[2 * m + 8]; v[2] = wd[2 * m + 1]; v[3] = wd[2 * m + 9];
            *reinterpret_cast<uintx4*>(dst + 16 * m) = v;
          }
        }
      } else if (OUT && p.codes && valid) {
#pragma unroll
        for (int f4 = 0; f4 < L / 8; ++f4) {
          const int f = 4 * f4;
          const uint32_t pk = pack4(acc[f / 16][f % 16], acc[f / 16][f % 16 + 1], acc[f / 16][f % 16 + 2], acc[f / 16][f % 16 + 3]);
          const int j0 = 8 * f4 + 4 * h;
          if (AXIS == CAFEQ_AXIS_COL) {
            *reinterpret_cast<uint32_t*>(p.codes + line * p.cols + ax0 + j0) = pk;
          } else {
            int8_t* rowp = p.codes + (ax0 + j0) * p.cols + line;
#pragma unroll
            for (int e = 0; e < 4; ++e) rowp[int64_t(e) * p.cols] = int8_t(pk >> (8 * e));
          }
        }
      }
      return NB == 1 ? dsc * dsc : usc2;
    };

    // ---- the phases of this run of n macro-tiles: strip m = matrix phase (inverse transform of strip m-1,
    // forward transform of strip m), barrier, vector phase (epilogue of strip m), barrier; one more matrix
    // phase for the last strip's inverse transform.  Group 1 runs one phase behind group 0: it waits one barrier
    // before its first phase, group 0 one after its last.  The first and the last phase are written out
    // separately so that inside the loop every register array is defined and consumed in the same iteration.
    //
    // Phase fences.  The compiler may move register-only work across a barrier; the empty asm statements take a
    // phase's results as in-out operands, so that everything that produces them stays before the barrier and
    // everything that consumes them after it (the scale factor included: the wait for its load belongs to the
    // matrix phase, so that the vector phase never waits on the memory counter; the running sum of the inverse phase too,
    // whose 64 multiply-adds belong into the shadow of its products and not into the vector phase).
    auto fence_m = [&]() {
      asm volatile("" : "+v"(usc), "+v"(s_l2), "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));
      __builtin_amdgcn_s_barrier();
    };
    auto fence_v = [&]() {
      asm volatile("" : "+v"(ebf[0]), "+v"(ebf[1]), "+v"(ebf[2]), "+v"(ebf[3]), "+v"(ebf[4]), "+v"(ebf[5]), "+v"(ebf[6]),
                   "+v"(ebf[7]), "+v"(ebf[8]), "+v"(ebf[9]), "+v"(ebf[10]), "+v"(ebf[11]), "+v"(ebf[12]), "+v"(ebf[13]),
                   "+v"(ebf[14]), "+v"(ebf[15]));
      asm volatile("" : "+v"(ebf[16]), "+v"(ebf[17]), "+v"(ebf[18]), "+v"(ebf[19]), "+v"(ebf[20]), "+v"(ebf[21]),
                   "+v"(ebf[22]), "+v"(ebf[23]), "+v"(ebf[24]), "+v"(ebf[25]), "+v"(ebf[26]), "+v"(ebf[27]), "+v"(ebf[28]),
                   "+v"(ebf[29]), "+v"(ebf[30]), "+v"(ebf[31]), "+v"(usc2_prev));
      if constexpr (EP == 2) {
#pragma unroll
        for (int i = 0; i < L / 4; i += 8)
          asm volatile("" : "+v"(elo[i]), "+v"(elo[i + 1]), "+v"(elo[i + 2]), "+v"(elo[i + 3]), "+v"(elo[i + 4]), "+v"(elo[i + 5]),
                       "+v"(elo[i + 6]), "+v"(elo[i + 7]));
      }
      __builtin_amdgcn_s_barrier();
    };
    if (grp == 1) __builtin_amdgcn_s_barrier();
    {
      if constexpr (!EARLY) request_strip(seg, int64_t(mis0) * kV2Waves + wave);
      rescale_strip(seg, int64_t(mis0) * kV2Waves + wave);
      forward();
      usc = __uint_as_float(__float_as_uint(lsc_nx) & 0x7F800000u) * fsc;   // (without the marks)
      fence_m();
      if constexpr (EARLY) request_next(0);
      usc2_prev = epilogue(0);
      fence_v();
    }
    for (int m = 1; m < n; ++m) {
      // The matrix phase wins the issue arbitration on its SIMD: its MFMAs go out as soon as the matrix pipe is
      // free and the other wave's vector phase fills the issue slots in between (at equal priority the vector
      // stream crowds out the first part of this phase and then leaves the rest of it without company).
      if constexpr (!EARLY) request_strip(seg, int64_t(mis0 + m) * kV2Waves + wave);
      __builtin_amdgcn_s_setprio(3);
      inverse(usc2_prev);
      rescale_strip(seg, int64_t(mis0 + m) * kV2Waves + wave);
      forward();
      __builtin_amdgcn_s_setprio(0);
      usc = __uint_as_float(__float_as_uint(lsc_nx) & 0x7F800000u) * fsc;   // (without the marks)
      fence_m();
      if constexpr (EARLY) request_next(m);
      usc2_prev = epilogue(m);
      fence_v();
    }
    inverse(usc2_prev);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_s_barrier();
    if (grp == 0) __builtin_amdgcn_s_barrier();

    // ---- publish this (workgroup, segment) partial: per-lane sums -> waves -> workgroup
    {
      const int64_t slot = w + seg;
      float vals[kHdrVa2 + NGRP];
      vals[kHdrL2] = s_l2; vals[kHdrErrZ] = s_errz; vals[kHdrWsq] = 0.f; vals[kHdrSur] = s_sur;
      vals[kHdrMref] = 0.f; vals[5] = 0.f; vals[6] = 0.f; vals[7] = 0.f;
#pragma unroll
      for (int i = 0; i < NGRP; ++i) vals[kHdrVa2 + i] = s_va2[i];
#pragma unroll
      for (int i = 0; i < kHdrVa2 + NGRP; ++i) {
        const float t = wave_sum(vals[i]);
        if (lane == 0) hred[wave * kHdrFloats + i] = t;
      }
      if (lane == 0) hred[wave * kHdrFloats + kHdrMref] = m_ref;
      __syncthreads();
      if (tid < kHdrVa2 + NGRP) {
        float t = 0.f;
        if (tid == kHdrMref || (tid == kHdrSur && lse_on)) {
          // waves keep their own references: rescale their sums of exponentials to the largest
          float mm = -INFINITY;
#pragma unroll
          for (int ww = 0; ww < kV2Waves; ++ww) mm = fmaxf(mm, hred[ww * kHdrFloats + kHdrMref]);
          if (tid == kHdrMref) {
            t = mm;
          } else {
#pragma unroll
            for (int ww = 0; ww < kV2Waves; ++ww) {
              const float sw = hred[ww * kHdrFloats + kHdrSur];
              if (sw > 0.f) t += sw * __expf(p.lse_t * (hred[ww * kHdrFloats + kHdrMref] - mm));
            }
          }
        } else {
#pragma unroll
          for (int ww = 0; ww < kV2Waves; ++ww) t += hred[ww * kHdrFloats + tid];
        }
        if (tid == kHdrWsq && wsq_pending) t = *p.prep_wsq;
        p.slot_hdr[slot * kHdrFloats + tid] = t;
      }
      wsq_pending = false;
      __syncthreads();
      s_l2 = s_errz = s_sur = 0.f;
      m_ref = -INFINITY;
#pragma unroll
      for (int i = 0; i < NGRP; ++i) s_va2[i] = 0.f;
    }
    mt += n;
  }
  if constexpr (SELF) {
    // a range that ends with its segment leaves the header behind its last one to nobody (workgroup w + 1 begins a segment
    // further): it must read as empty (otherwise the planes' launch resets the headers)
    const int last = int((mt1 - 1) / mt_per_seg);
    if (mt1 == int64_t(last + 1) * mt_per_seg && tid < kHdrFloats)
      p.slot_hdr[(w + last + 1) * kHdrFloats + tid] = tid == kHdrMref ? -INFINITY : 0.f;
  }
}

template <int K, int G, int AXIS, bool REC, bool OUT, int WP>
__global__ __launch_bounds__(kV2Threads, 1) void loss_v2_kernel(const CoreParams p) {
  loss_v2_body<K, G, AXIS, REC, OUT, WP, v2_splits_planes(K, false, OUT), false>(p, blockIdx.x);
}

// Both members of a pair in one launch (no codes or scales requested): the first pa.nwg workgroups take member
// A, the others member B.  With one workgroup per compute unit in total, half of the chip streams each member
// and the ranges of the two members end together -- one kernel tail instead of two.
// WPA, WPB: parts of the members' weights.
template <int K, int G, bool REC, int WPA, int WPB>
__global__ __launch_bounds__(kV2Threads, 1) void loss_v2_pair_kernel(const CoreParams pa, const CoreParams pb) {
  constexpr bool SELF = v2_splits_planes(K, true, false);
  if (blockIdx.x < unsigned(pa.nwg)) loss_v2_body<K, G, CAFEQ_AXIS_COL, REC, false, WPA, SELF, true>(pa, blockIdx.x);
  else loss_v2_body<K, G, CAFEQ_AXIS_ROW, REC, false, WPB, SELF, true>(pb, blockIdx.x - unsigned(pa.nwg));
}

template <int K, int G, int AXIS, bool REC, bool OUT, int WP>
int launch_v2_v(const CoreParams& p, hipStream_t st) {
  auto kern = loss_v2_kernel<K, G, AXIS, REC, OUT, WP>;
  static std::atomic<bool> attr_set{false};   // per instantiation
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024) != hipSuccess)
      return CAFEQ_ERR_LAUNCH;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3(unsigned(p.nwg)), dim3(kV2Threads), v2_lds(K), st, p);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
template <int K, int G, int AXIS, int WP>
int launch_v2_p(const CoreParams& p, hipStream_t st) {
  if (p.codes || p.scales)
    return p.rec ? launch_v2_v<K, G, AXIS, true, true, WP>(p, st) : launch_v2_v<K, G, AXIS, false, true, WP>(p, st);
  return p.rec ? launch_v2_v<K, G, AXIS, true, false, WP>(p, st) : launch_v2_v<K, G, AXIS, false, false, WP>(p, st);
}
template <int K, int G, int AXIS>
int launch_v2_t(const CoreParams& p, hipStream_t st) {
  return prepared_parts(p.dtype) == 1 ? launch_v2_p<K, G, AXIS, 1>(p, st) : launch_v2_p<K, G, AXIS, 2>(p, st);
}

template <int K, int G, bool REC, int WPA, int WPB>
int launch_v2_pair_w(const CoreParams& pa, const CoreParams& pb, hipStream_t st) {
  auto kern = loss_v2_pair_kernel<K, G, REC, WPA, WPB>;
  static std::atomic<bool> attr_set{false};   // per instantiation
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024) != hipSuccess)
      return CAFEQ_ERR_LAUNCH;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3(unsigned(pa.nwg + pb.nwg)), dim3(kV2Threads), v2_lds(K), st, pa, pb);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
template <int K, int G, bool REC>
int launch_v2_pair_v(const CoreParams& pa, const CoreParams& pb, hipStream_t st) {
  const bool oa = prepared_parts(pa.dtype) == 1, ob = prepared_parts(pb.dtype) == 1;
  if (oa) return ob ? launch_v2_pair_w<K, G, REC, 1, 1>(pa, pb, st) : launch_v2_pair_w<K, G, REC, 1, 2>(pa, pb, st);
  return ob ? launch_v2_pair_w<K, G, REC, 2, 1>(pa, pb, st) : launch_v2_pair_w<K, G, REC, 2, 2>(pa, pb, st);
}

template <int K>
int launch_v2_pair_k(int G, const CoreParams& pa, const CoreParams& pb, hipStream_t st) {
  const bool rec = pa.rec != nullptr;
  switch (G) {
    case 32: return rec ? launch_v2_pair_v<K, 32, true>(pa, pb, st) : launch_v2_pair_v<K, 32, false>(pa, pb, st);
    case 64: return rec ? launch_v2_pair_v<K, 64, true>(pa, pb, st) : launch_v2_pair_v<K, 64, false>(pa, pb, st);
    case 128: return rec ? launch_v2_pair_v<K, 128, true>(pa, pb, st) : launch_v2_pair_v<K, 128, false>(pa, pb, st);
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
}
template <int K>
int launch_v2_k(int G, int axis, const CoreParams& p, hipStream_t st) {
  const bool col = axis == CAFEQ_AXIS_COL;
  switch (G) {
    case 32: return col ? launch_v2_t<K, 32, CAFEQ_AXIS_COL>(p, st) : launch_v2_t<K, 32, CAFEQ_AXIS_ROW>(p, st);
    case 64: return col ? launch_v2_t<K, 64, CAFEQ_AXIS_COL>(p, st) : launch_v2_t<K, 64, CAFEQ_AXIS_ROW>(p, st);
    case 128: return col ? launch_v2_t<K, 128, CAFEQ_AXIS_COL>(p, st) : launch_v2_t<K, 128, CAFEQ_AXIS_ROW>(p, st);
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
}

}  // namespace
}  // namespace cafeq
