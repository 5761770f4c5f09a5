// extern "C" entry points: argument validation and dispatch.  See include/cafeq.h.
#include <utility>
#include <vector>

#include "xform_core.hpp"
#include "loss_reduce.hpp"
#include "mmid.hpp"

using namespace cafeq;
namespace cafeq {
// (defined further down, next to the timing table)
int launch_grad_owner_timed(const GradOwnerJob* jobs, int n, int loss_kind, float beta, float lse_t, const double* lse_ms,
                            hipStream_t st, const LossArgs* fold);
int launch_grad_v2_timed(const CoreParams& p, hipStream_t st);
int launch_core32_timed(int axis, const CoreParams& p, hipStream_t st);
int launch_grad_pass_timed(int K, int axis, const CoreParams& p, hipStream_t st);
int launch_grad_gather_timed(int K, const GradGatherJob* jobs, int n, const LossArgs& la, const VArgs* va, hipStream_t st,
                             const RhoGroups* rho = nullptr);
}  // namespace cafeq

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_mat(const cafeq_mat* m) {
  if (!m || !m->data) return CAFEQ_ERR_INVALID_ARG;
  if (m->dtype != CAFEQ_F32 && m->dtype != CAFEQ_BF16) return CAFEQ_ERR_INVALID_ARG;
  if (m->rows <= 0 || m->cols <= 0 || m->ld < m->cols) return CAFEQ_ERR_BAD_SHAPE;
  if (m->cols % 4 != 0) return CAFEQ_ERR_BAD_SHAPE;
  const int64_t ldm = m->dtype == CAFEQ_F32 ? 4 : 8;
  if (m->ld % ldm != 0 || !aligned16(m->data)) return CAFEQ_ERR_BAD_ALIGN;
  return CAFEQ_OK;
}

// allow_minmax: the call has kernels for the min/max grid of Eq. (1)
int check_cfg(const cafeq_quant_cfg* c, bool need_axis, bool allow_minmax = false) {
  if (!c) return CAFEQ_ERR_INVALID_ARG;
  if (c->bits < 2 || c->bits > 8 || c->group < 0) return CAFEQ_ERR_INVALID_ARG;
  if (need_axis && c->axis != CAFEQ_AXIS_COL && c->axis != CAFEQ_AXIS_ROW) return CAFEQ_ERR_INVALID_ARG;
  if (c->mode == CAFEQ_Q_ASYM_MINMAX) return allow_minmax ? CAFEQ_OK : CAFEQ_ERR_UNSUPPORTED;
  if (c->mode != CAFEQ_Q_SYM_ABSMAX) return CAFEQ_ERR_INVALID_ARG;
  return CAFEQ_OK;
}


// ---------------------------------------------------------------------------------------
// planning of one fused-core launch and its scratch layout
// ---------------------------------------------------------------------------------------
struct CorePlan {
  int K, G, L, NBLK, NGRP, nseg, nwg;
  int64_t nlines, naxis, mt_per_seg, n_mt, nslot;
  size_t slot_grad_floats;   // per slot
};

bool supported_block(int k) { return k == 32 || k == 64 || k == 128 || k == 256; }

// How the quantization groups of one matrix lie over the fused core's segments.  Groups of 32, 64, 128 or
// 256 are a compile-time parameter of the core (a segment holds whole groups).  Any longer group -- a whole
// channel, the per-channel setting of the paper's experiments, included -- spans `gspan` segments of `Gk`
// elements; the core then runs with one group per segment and the group's absmax is assembled from the
// segments' records (CoreParams::gspan).
struct GroupPlan {
  int G;       // group length along the axis
  int Gk;      // the core's compile-time group
  int gspan;   // segments per group
};
int resolve_group(const cafeq_quant_cfg* cfg, int64_t naxis, int K, GroupPlan* gp) {
  const int64_t g = cfg->group == 0 ? naxis : cfg->group;
  if (g <= 0 || naxis % g != 0) return CAFEQ_ERR_BAD_SHAPE;
  if (g > (int64_t(1) << 30)) return CAFEQ_ERR_UNSUPPORTED;
  gp->G = int(g);
  if (g == 32 || g == 64 || g == 128 || g == 256) { gp->Gk = int(g); gp->gspan = 1; return CAFEQ_OK; }
  int L = K > 128 ? K : 128;
  if (g % L != 0) L = K;
  if (g < L || g % L != 0) return CAFEQ_ERR_UNSUPPORTED;
  gp->Gk = L; gp->gspan = int(g / L);
  return CAFEQ_OK;
}

// Workgroups for n macro-tiles on `slots` places: one each while they fit, else a multiple of eight (ranges that follow each other then
// sit behind one L2).  Down to a multiple of eight in either case, a few tiles were left for a second round.
// Evaluations, us: 1152 x 1152 76 / 71, 300 x 1152 75 / 66, pairs 300 x 1664 76 / 67, at k = 256 2304 x 2304 329 / 282; whole channels 700 x 3328 99 / 92.
int workgroups(int64_t n, int64_t slots) { return int(n <= slots || slots <= 8 ? std::min(n, slots) : slots - slots % 8); }

// grad: the launch will ask for the fused gradient.  Without it, segments of up to 128 run two
// workgroups per compute unit; segments of 32 do in either case.
int make_plan(int K, int G, int64_t nlines, int64_t naxis, CorePlan* pl, bool grad = true) {
  if (!supported_block(K)) return CAFEQ_ERR_UNSUPPORTED;
  if (!(G == 32 || G == 64 || G == 128 || G == 256)) return CAFEQ_ERR_UNSUPPORTED;
  pl->K = K; pl->G = G; pl->L = K > G ? K : G;
  if (naxis % pl->L != 0) return CAFEQ_ERR_BAD_SHAPE;
  pl->NBLK = pl->L / K; pl->NGRP = pl->L / G;
  pl->nlines = nlines; pl->naxis = naxis;
  pl->nseg = int(naxis / pl->L);
  pl->mt_per_seg = (nlines + kMacroLines - 1) / kMacroLines;
  pl->n_mt = pl->mt_per_seg * pl->nseg;
  const int per_cu = pl->L == 32 || (!grad && pl->L <= 128) ? 2 : 1;
  pl->nwg = workgroups(pl->n_mt, int64_t(device_cu_count()) * per_cu);
  pl->nslot = pl->nwg + pl->nseg;
  pl->slot_grad_floats = size_t(pl->NBLK) * K * K;
  return CAFEQ_OK;
}

// The gradient pass of the two-pass scheme walks the axis in chunks of 128 inputs, two workgroups per
// compute unit (one for blocks of 256).
int make_grad_plan(int K, int64_t nlines, int64_t naxis, CorePlan* pl) {
  if (!supported_block(K)) return CAFEQ_ERR_UNSUPPORTED;
  if (naxis % 128 != 0) return CAFEQ_ERR_UNSUPPORTED;
  pl->K = K; pl->G = 0; pl->L = 128; pl->NBLK = 0; pl->NGRP = 0;
  pl->nlines = nlines; pl->naxis = naxis;
  pl->nseg = int(naxis / 128);
  pl->mt_per_seg = (nlines + kMacroLines - 1) / kMacroLines;
  pl->n_mt = pl->mt_per_seg * pl->nseg;
  int64_t nwg = std::min<int64_t>(pl->n_mt, int64_t(device_cu_count()) * (K == 256 ? 1 : 2));
  if (nwg > 8) nwg -= nwg % 8;
  // A whole number of workgroups per chunk, where the longest range gets no longer by it: no range then
  // straddles two chunks (one partial per workgroup instead of up to two) and all ranges are equal.
  {
    const int64_t per = nwg / pl->nseg;
    if (per >= 1 && pl->mt_per_seg % per == 0 && pl->mt_per_seg / per <= (pl->n_mt + nwg - 1) / nwg &&
        (per * pl->nseg) % 8 == 0)
      nwg = per * pl->nseg;
  }
  pl->nwg = int(nwg);
  pl->nslot = pl->nwg + pl->nseg;
  pl->slot_grad_floats = grad_pass_part_floats(K);
  return CAFEQ_OK;
}

struct Carver {
  char* base; size_t off;
  explicit Carver(void* b) : base(static_cast<char*>(b)), off(0) {}
  template <typename T> T* take(size_t n) {
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off = align_up(off + n * sizeof(T), 256);
    return p;
  }
};

// Whether the loss pass for (K, G) runs its forward contraction on two-part half-precision operands: the
// gradient-free kernel variant over 128 x 128 blocks with one block per segment, for grids of up to 4 bits
// (two float16 parts carry 22 of float32's 24 bits; the error that leaves in z / scale grows with the number of
// levels, so finer grids keep the six-product bfloat16 forward).
bool core_forward_f16(int K, int G, int bits) { return K == 128 && G <= 128 && bits <= 4; }

// Plans of one matrix for a call with / without gradient: `first` is the pass that computes the losses,
// `gpass` the pass that writes the gradient partials (== first when the gradient is fused into it).
// The gradient runs as a second pass over the weights, from the loss pass's arg-max records, where the fused
// kernel has no gradient (blocks of 256, groups of 256 with blocks of 64 or more), where the two passes are
// faster (blocks of 128), and for groups that span several segments.
// asym: the min/max grid of Eq. (1); its kernel variants are gradient-free, so the gradient always takes the
// second pass.
struct PassPlans { CorePlan first, gpass; GroupPlan gp; bool two, fused, v2, asym, gather, core32; };
bool is_minmax(const cafeq_quant_cfg* cfg) { return cfg->mode == CAFEQ_Q_ASYM_MINMAX; }
// levels and the surrogate's constant for either grid (Sec. 4.1: 1 / (2^b - 1)^2 for Eq. (1); a quarter of the
// squared step of the symmetric grid)
QGrid grid_for(const cafeq_quant_cfg* cfg) {
  if (!is_minmax(cfg)) return make_grid(cfg->bits);
  QGrid g;
  g.qmax = float((1 << cfg->bits) - 1);
  g.qmin = 0.f;
  return g;
}
float beta_for(const cafeq_quant_cfg* cfg, const QGrid& g) {
  return is_minmax(cfg) ? 1.f / (g.qmax * g.qmax) : 1.f / (4.f * g.qmax * g.qmax);
}
// The loss pass over prepared weights (loss_v2.hip): one workgroup of eight waves per compute unit,
// macro-tiles of 256 lines.
// codes_along_rows: it writes codes or scales of a matrix transformed along its rows (byte stores).  Blocks of 32 and 64 with
// float32 weights have no registers for that next to two parts of everything: 9216 x 2304, groups of 32 and 64 48 to 58 us
// the general way (k = 32 with groups of 32 in its own kernel 39), 58 to 69 this way; groups of 128 54 and 56 at k = 32, 58 and 50 at k = 64.
bool v2_eligible(const cafeq_mat* W, int K, const GroupPlan& gp, const cafeq_quant_cfg* cfg, bool codes_along_rows) {
  if (K < 128 && codes_along_rows && W->dtype == CAFEQ_F32 && !(K == 64 && gp.Gk == 128)) return false;
  return W->prepared != nullptr && K <= 128 && gp.Gk <= 128 && gp.gspan == 1 && cfg->bits <= 4 && !is_minmax(cfg);
}
// share: the matrix gets 1 / share of the chip's compute units (2: the members of a pair that run in one launch)
void make_v2_plan(CorePlan* pl, int share = 1) {
  // (segments of 128 whatever the block)
  pl->L = 128; pl->NBLK = 128 / pl->K; pl->NGRP = 128 / pl->G; pl->nseg = int(pl->naxis / 128);
  pl->mt_per_seg = (pl->nlines + 255) / 256;
  pl->n_mt = pl->mt_per_seg * pl->nseg;
  pl->nwg = workgroups(pl->n_mt, int64_t(device_cu_count()) / share);
  pl->nslot = pl->nwg + pl->nseg;
}
// rounds of workgroups that the loss pass takes over prepared weights and in the general kernel, in multiples of eight, as both ran when
// the lines below were drawn (k = 32 with groups of 32 has had a kernel of its own since, core32.hip, in the general one's place: figures at the
// lines).  Both now take a workgroup a tile while they fit (workgroups()): more than eight tiles that are no multiple of
// eight count as two rounds here and run as one.  Timed again over 9600 shapes of 32 to 36864 lines, launches replayed from a graph, the
// choices below lose against the faster pass of each shape, on average: without codes 0.2 to 4 % at k = 32 and 2 to 6 at 64 (most with groups
// of 32 and 64: prepared / general .92 in bfloat16, 1.05 in float32 for 65 to 256 tiles of the general kernel, .77 and .90 up to 512); pairs 0 to 4, in float32 at k = 64
// 9; with codes 1 to 12; and 10 to 26 with bfloat16 codes along rows, which the general kernel writes faster at every size (1.1 to 2).
bool v2_rounds(int K, int G, int64_t nlines, int64_t naxis, int share, int64_t* here, int64_t* there) {
  CorePlan pl;
  if (make_plan(K, G, nlines, naxis, &pl, false)) return false;
  auto rounds = [&]() {
    const int64_t nwg = pl.nwg > 8 ? pl.nwg - pl.nwg % 8 : pl.nwg;
    return (pl.n_mt + nwg - 1) / nwg;
  };
  *there = rounds();
  make_v2_plan(&pl, share);
  *here = rounds();
  return true;
}
// Whether the loss pass over prepared weights is the faster one (blocks of 128: always; blocks of 32 and 64: not where there
// are few of its tiles).  Both kernels take as long as their rounds of workgroups do: one a compute unit and tiles of 256 lines x
// 128 indices here, two a unit and 128 lines x one segment of max(K, G) indices there.  Losses alone, the general kernel's
// time / this one's in us, at k = 64: 1152 x 512 (two rounds here, one there), groups of 64 13 / 20; 2304 x 2304 (two and two),
// groups of 64 21 / 21, of 128 31 / 20; 36864 x 4608 (21 and 41) 293 / 178.
bool v2_pays(const cafeq_mat* W, int K, const GroupPlan& gp, int64_t nlines, int64_t naxis, bool out, bool along_rows) {
  if (K == 128) return true;
  int64_t here, there;
  if (!v2_rounds(K, gp.Gk, nlines, naxis, 1, &here, &there)) return false;
  const bool bf16 = W->dtype == CAFEQ_BF16, more = here > 1;
  // (two tiles of 256 for 304 lines: 304 x 36864 at k = 32, groups of 64 44 / 50, in bfloat16 46 / 44)
  if (K == 32 && !bf16 && 2 * ((nlines + 255) / 256 * 256) > 3 * nlines) return false;
  switch (std::max(K, gp.Gk)) {
    case 128: return there >= 1 + int(more || (out && along_rows && !bf16));
    case 64: return there >= 2 + int(more && (K == 32 || !bf16 || out || nlines < 512));
    // (k = 32 with groups of 32, a line drawn against the general kernel and not redrawn against core32.hip, which takes the other side's place:
    // it is the faster one further up, to about 50 M weights in float32 and 10 to 20 M in bfloat16, with codes further still.  core32 / this one, us, by
    // replayed graphs, in bfloat16 behind the semicolon: losses 1152 x 512 7.8 / 19; 7.9 / 17, 2304 x 2304 15 / 22; 15 / 18.5, 2304 x 9216 36 / 45; 35.7 / 37.3,
    // 9216 x 2304 33 / 42; 33 / 33.6, 3584 x 14336 69 / 67; 67 / 56, 36864 x 4608 214 / 180; 216 / 134; with codes along columns 2304 x 9216 42 / 59; 41 / 72,
    // 3584 x 14336 109 / 108; 79 / 128, 36864 x 4608 411 / 279; 426 / 426, along rows in bfloat16 39 / 82, 79 / 144 and 251 / 399)
    default: return there >= (bf16 && !(out && along_rows) ? 3 + int(more) : 3 * here + 1);
  }
}
// The same for a pair whose members share a launch, half of the chip each, against two launches: at k = 32, groups of 32 (core32.hip the other
// side) 600 x 512 13.5 / 20.2, 3584 x 512 17.2 / 20.7, 4608 x 1024 30.4 / 28.7, 3584 x 4096 50 / 43, 3584 x 14336 153 / 121, in bfloat16 13.8 / 18.5, 17.3 / 18.8,
// 27.7 / 24.3, 49 / 36 and 139 / 90; groups of 64 256 x 2304 22 / 28, else from 22 / 22 down.
bool v2_pair_pays(const cafeq_mat* A, const cafeq_mat* B, int K, const GroupPlan& gp) {
  if (std::max(K, gp.Gk) == 128) return true;
  int64_t ha, ta, hb, tb;
  if (!v2_rounds(K, gp.Gk, A->rows, A->cols, 2, &ha, &ta) || !v2_rounds(K, gp.Gk, B->cols, B->rows, 2, &hb, &tb)) return false;
  const bool few = ha + hb > 2, bf16 = A->dtype == CAFEQ_BF16 && B->dtype == CAFEQ_BF16;
  if (std::max(K, gp.Gk) == 64) return (bf16 && K == 64) || ta + tb > 2 || !few;
  return ta + tb >= 2 + int(!bf16) + int(few);
}

// Whether the gradient can come from the arg-max records by gathering lines (grad_gather.hip): a line's inputs lie side by
// side (columns, or rows with the prepared line-major copy) and a block meets one group per line, or is one of 256, whose
// product with the matrix of zeros (grad_core.hpp) runs one wave per SIMD.  Gradient passes with their reductions, product /
// by records: 9B-shaped pair (blocks of 128) 97 / 90 us, 27B-shaped in bfloat16 246 / 165, 2B-shaped 59 / 42; 2304 x 9216
// whole channels 48 / 16; 9B-shaped (V, O) pair, blocks of 256 and groups of 64, whose lines are read four times, 99 / 70.
// Blocks of 128 with groups of 64 would read every line twice: 97 / about 150.
bool gather_possible(int K, const GroupPlan& gp, bool lines) { return lines && (gp.G >= K || K == 256); }
// Whether that is the faster way.  A workgroup sorts the records of one block (of a block's group where those are shorter), so that
// few blocks of many lines leave the chip to a few workgroups, where the product spreads over lines as well.  Whole
// evaluations in us, the other way / by records:
//   groups from 128 on at k = 256, longer than 128 elsewhere: by records throughout (36864 x 256 at k = 256 205 / 190; whole channels
//   at k = 128 159 / 136).  k = 256, groups of 64 (every line four times): 36864 x 1024 357 / 360, x 256 204 / 215; groups of 32 (eight
//   times): 4608 x 1024 132 / 121, 2304 x 4608 .99, and with a block's lines behind one L2 2304 x 9216 478 / 454 (inverse and all), pairs
//   3584 x 4096 425 / 381, 4608 x 14336 1274 / 1486; 36864 x 4608 1384 / 1671, in bfloat16 1387 / 1280.
//   k = 128, groups of 128: 14336 x 1024 .97, 36864 x 256 118 / 110, x 1024 164 / 171, x 4608 580 / 507, and with prepared weights, whose product
//   reads tiles in its own order, 127 / 142 and 385 / 393.
//   k = 32 with groups of 32, whose loss pass (core32.hip) forms the gradient on its way, as exact: single matrices on the way at every size
//   (by records / on the way, launches replayed from a graph, without the inverse: 4104 x 2048 43 / 29, 4888 x 2048 48 / 30, 1152 x 9216 49 / 31,
//   304 x 36864 67 / 45, prepared 2304 x 9216 87 / 48, in bfloat16 78 / 47; with it 36864 x 2304 282 / 151, 4608 x 36864 447 / 291), but for large
//   ones in bfloat16 along rows, of which a wave asks for 64 bytes at a time: 4888 x 2048 55 / 32, 36864 x 1024 167 / 103, 3584 x 14336 132.7 / 133.2,
//   36864 x 4608 349 / 479.  Pairs in float32 from 1 M weights a member on (1000 x 4096 80 / 57, 3584 x 14336 270 / 208; below either way does:
//   136 x 512 22.4 / 22.2, 1024 x 512 24.8 / 23.3, 1152 x 1024 27.5 / 27.5); in bfloat16 by records (1000 x 4096 42.5 / 38.5, 3584 x 14336 224 / 233, with
//   the inverse 2304 x 9216 116 / 125, 4608 x 36864 648 / 809).
//   Other groups at k = 32 and 64 in one matrix, where the general loss pass forms the gradient on its way: 14336 x 1024 (k = 32) 68 / 85, 36864 x 2304
//   308 / 259, 2304 x 4608 58 / 55, 1147 x 9216 63 / 61, 4.2 M weights 33 / 40; over prepared weights, whose loss pass only records, with groups of 128
//   (bfloat16: of 64) 36864 x 1024 113 / 107, 9216 x 1024 57 / 50.  On the min/max grid, a pass of its own either way: groups of 32 1147 x 512
//   31 / 25, 4608 x 256 33 / 37, 2304 x 9216 83 / 86, 36864 x 1024 120 / 184; 64 36864 x 1024 118 / 140, 14336 x 512 66 / 61.
//   Pairs (prepared: two launches less): 4608 x 256 at k = 32, groups of 32 48 / 56, 2304 x 512 47 / 46; else by records throughout.
bool gather_pays(const cafeq_mat* W, int K, const GroupPlan& gp, int64_t nlines, int64_t naxis, bool asym, bool pair, bool v2, bool along_rows) {
  const int64_t weights = nlines * naxis;
  const bool bf16 = W->dtype == CAFEQ_BF16;
  if (K == 32 && gp.G == 32 && !asym && (pair ? !bf16 && weights >= int64_t(1) << 20 : !(bf16 && along_rows) || weights < 50000000)) return false;
  const bool on_the_way = !pair && K <= 64 && gp.gspan == 1 && core_lds_bytes(K, gp.Gk, true) != 0 && !asym;
  if (on_the_way && weights < (int64_t(1) << 23)) return false;
  if (K == 256 && gp.G == 64) return bf16 || nlines <= 64 * naxis;
  if (K == 256 && gp.G == 32) return bf16 ? nlines <= 36 * naxis : nlines <= 24 * naxis && weights < 24000000;
  if (K == 256 || gp.G > 128 || gp.gspan > 1) return true;
  if (K == 128) return nlines <= 16384 || naxis <= 256 || (!W->prepared && naxis >= 2048);
  if (pair) return asym || gp.G > 32 || nlines <= 6 * naxis;
  if (asym) {
    if (gp.G == 32) return (nlines <= 2304 && naxis <= 4608) || (nlines <= 8192 && weights >= 64000000);
    return gp.G == 128 || nlines <= 30 * naxis;
  }
  if (v2 && (gp.G == 128 || (gp.G == 64 && bf16))) return naxis >= 1024;
  return naxis >= 2048 && weights >= 10000000;
}
bool has_lines(const cafeq_mat* W, int axis) {
  if (axis == CAFEQ_AXIS_COL) return grad_gather_fits(W->rows, W->ld, 128, W->dtype);
  return W->prepared && grad_gather_fits(W->cols, 128, prepared_layout(W->cols, W->rows, W->dtype, axis).nlp * 128, W->dtype);
}
int plan_passes(int K, const GroupPlan& gp, int64_t nlines, int64_t naxis, bool grad, PassPlans* pp,
                bool v2 = false, bool asym = false, int v2_share = 1, bool gather = false) {
  pp->gp = gp;
  pp->v2 = v2;
  pp->asym = asym;
  const size_t fl = core_lds_bytes(K, gp.Gk, true);
  const bool fused_ok = fl != 0 && fl <= 160 * 1024 && gp.gspan == 1 && !(K == 128 && gp.Gk <= 128) && !asym;
  pp->gather = grad && gather;
  pp->core32 = K == 32 && gp.G == 32 && !v2 && !asym;   // (a kernel of its own, which needs no prepared planes: core32.hip)
  pp->two = grad && (!fused_ok || gather);
  pp->fused = grad && fused_ok && !gather;
  int rc = make_plan(K, gp.Gk, nlines, naxis, &pp->first, pp->fused);
  if (rc) return rc;
  if (v2) make_v2_plan(&pp->first, v2_share);
  if (pp->two && !fused_ok && naxis % 128 != 0) return CAFEQ_ERR_UNSUPPORTED;
  if (pp->two && !pp->gather) return make_grad_plan(K, nlines, naxis, &pp->gpass);
  pp->gpass = pp->first;
  if (pp->gather) pp->gpass.nslot = 0;   // no partials
  return CAFEQ_OK;
}

// scratch of one matrix's passes
struct MemberWs {
  float *rG, *rGreal, *slot_grad, *fs, *fsi;
  uint16_t *pfwd, *pinv;
  float2 *rec, *grec;
  float2 *rec_mm, *grec_mm;   // min/max grid with groups that span segments
  float* zkeep;               // groups that span segments: the transformed weights between the sweeps
  uint2* sorted; int* start;  // gradient pass by records
};
size_t zkeep_floats(const PassPlans& pp) {
  const CorePlan& pl = pp.first;
  return pp.gp.gspan > 1 && pl.K >= kKeepBlock ? size_t(pl.n_mt) * kMacroLines * size_t(pl.L) : 0;
}
// zkeep: room for zkeep_floats(pp); members whose sweeps run one after the other share it
void carve_member(Carver& c, const PassPlans& pp, int nb, bool grad, bool want_rG, float* zkeep, MemberWs* w) {
  const CorePlan& pl = pp.first;
  const bool big = pp.gp.gspan > 1;
  w->fs = c.take<float>(nb);
  w->fsi = c.take<float>(nb);
  w->pfwd = c.take<uint16_t>(size_t(nb) * kFwdPlanes * pl.K * pl.K);
  w->pinv = c.take<uint16_t>(size_t(nb) * kInvPlanes * pl.K * pl.K);
  w->rG = c.take<float>(want_rG ? size_t(pl.naxis / pl.G) : 0);
  w->rGreal = big && want_rG ? c.take<float>(size_t(pl.naxis / pp.gp.G)) : w->rG;
  w->slot_grad = c.take<float>(grad ? size_t(pp.gpass.nslot) * pp.gpass.slot_grad_floats : 0);
  w->rec = c.take<float2>((pp.two || big) ? size_t(pl.naxis / pl.G) * size_t(pl.nlines) : 0);
  w->grec = big ? c.take<float2>(size_t(pl.naxis / pp.gp.G) * size_t(pl.nlines)) : w->rec;
  const bool mm = big && pp.asym;
  w->rec_mm = c.take<float2>(mm ? size_t(pl.naxis / pl.G) * size_t(pl.nlines) : 0);
  w->grec_mm = c.take<float2>(mm ? size_t(pl.naxis / pp.gp.G) * size_t(pl.nlines) : 0);
  if (!mm) w->rec_mm = w->grec_mm = nullptr;
  w->zkeep = zkeep_floats(pp) ? zkeep : nullptr;
  w->sorted = c.take<uint2>(pp.gather ? grad_gather_entries(pl.K, pp.gp.G, pl.naxis, pl.nlines) : 0);
  w->start = c.take<int>(pp.gather ? grad_gather_starts(pl.K, pp.gp.G, pl.naxis) : 0);
}

struct SingleWs {
  double* lse_ms; float* member_ref; float *rho, *slot_hdr, *mmid, *x1; MemberWs m; size_t bytes;
};
SingleWs carve_single(void* ws, const PassPlans& pp, int nb, bool grad) {
  Carver c(ws);
  SingleWs w;
  const CorePlan& pl = pp.first;
  w.lse_ms = c.take<double>(2);
  w.member_ref = c.take<float>(4);
  w.rho = c.take<float>(size_t(nb) * pl.K);
  w.slot_hdr = c.take<float>(size_t(pl.nslot) * kHdrFloats);
  w.mmid = c.take<float>(grad ? size_t(nb) * pl.K * pl.K : 0);
  w.x1 = c.take<float>(grad ? size_t(nb) * pl.K * pl.K : 0);
  carve_member(c, pp, nb, grad, true, c.take<float>(zkeep_floats(pp)), &w.m);
  w.bytes = c.off;
  return w;
}

struct DualWs {
  double* lse_ms; float* member_ref; float *hdrA, *hdrB, *gp, *x1; MemberWs a, b; size_t bytes;
};
DualWs carve_dual(void* ws, const PassPlans& qa, const PassPlans& qb, int nb, bool grad) {
  Carver c(ws);
  DualWs w;
  const int K = qa.first.K;
  w.lse_ms = c.take<double>(2);
  w.member_ref = c.take<float>(4);   // [0]: member A, [1]: member B
  w.hdrA = c.take<float>(size_t(qa.first.nslot + qb.first.nslot) * kHdrFloats);   // A then B, contiguous
  w.hdrB = w.hdrA ? w.hdrA + size_t(qa.first.nslot) * kHdrFloats : nullptr;
  w.gp = c.take<float>(grad ? size_t(nb) * K * K : 0);
  w.x1 = c.take<float>(grad ? size_t(nb) * K * K : 0);
  float* zkeep = c.take<float>(std::max(zkeep_floats(qa), zkeep_floats(qb)));
  carve_member(c, qa, nb, grad, false, zkeep, &w.a);
  carve_member(c, qb, nb, grad, false, zkeep, &w.b);
  w.bytes = c.off;
  return w;
}

int check_xform(const cafeq_xform* x, bool need_inv) {
  if (!x || !x->T || (need_inv && !x->Tinv)) return CAFEQ_ERR_INVALID_ARG;
  if (!supported_block(x->k)) return CAFEQ_ERR_UNSUPPORTED;
  if (x->nb <= 0 || x->rep <= 0) return CAFEQ_ERR_BAD_SHAPE;
  if (!aligned16(x->T) || (x->Tinv && !aligned16(x->Tinv))) return CAFEQ_ERR_BAD_ALIGN;
  return CAFEQ_OK;
}

int check_axis_len(const cafeq_mat* W, const cafeq_xform* x, int axis) {
  if (axis == CAFEQ_AXIS_COL) {
    if (x->rep != 1 || W->cols != int64_t(x->nb) * x->k) return CAFEQ_ERR_BAD_SHAPE;
  } else if (axis == CAFEQ_AXIS_ROW) {
    if (W->rows != int64_t(x->nb) * x->rep * x->k) return CAFEQ_ERR_BAD_SHAPE;
  } else {
    return CAFEQ_ERR_INVALID_ARG;
  }
  return CAFEQ_OK;
}

// Transform blocks of 2, 4, 8 or 16: a run of 32 / k of them is one block-diagonal block of 32, which is how every
// entry point below runs them (embed into scratch, call itself with blocks of 32, gather the gradient's diagonal
// sub-blocks).  small_m: 32 / k for those sizes, 0 for any other.
int small_m(int k) { return (k == 2 || k == 4 || k == 8 || k == 16) ? 32 / k : 0; }
struct SmallWs { float *T32, *P32, *G32; int* st32; void* sub; size_t head; };
SmallWs carve_small(void* ws, int64_t nb32) {
  Carver c(ws);
  SmallWs w;
  w.T32 = c.take<float>(size_t(nb32) * 1024);
  w.P32 = c.take<float>(size_t(nb32) * 1024);
  w.G32 = c.take<float>(size_t(nb32) * 1024);
  w.st32 = c.take<int>(size_t(nb32));
  w.head = c.off;
  w.sub = ws ? static_cast<char*>(ws) + c.off : nullptr;
  return w;
}
// blocks of 32 that a small-block transform over `naxis` indices makes (0: not a whole number)
int64_t small_nb32(const cafeq_xform* x, int64_t naxis) {
  if (naxis % 32 != 0 || naxis != int64_t(x->nb) * x->rep * x->k) return 0;
  return naxis / 32;
}
int check_small_xform(const cafeq_xform* x, bool need_inv) {
  if (!x || !x->T || (need_inv && !x->Tinv)) return CAFEQ_ERR_INVALID_ARG;
  if (x->nb <= 0 || x->rep <= 0) return CAFEQ_ERR_BAD_SHAPE;
  if (!aligned16(x->T) || (x->Tinv && !aligned16(x->Tinv))) return CAFEQ_ERR_BAD_ALIGN;
  return CAFEQ_OK;
}
size_t orth_ws_any(int k, int nb) {
  if (!small_m(k)) return orth_workspace_bytes(k, nb);
  const int64_t nb32 = int64_t(nb) * k / 32;
  return carve_small(nullptr, nb32).head + orth_workspace_bytes(32, int(nb32));
}

struct AdaptivePlan {
  GroupPlan ga, gb;
  int nchunkA, nchunkB;
  int64_t chunkA, chunkB;
  CorePlan planU, planV;
  size_t partial_floats, rec_entries, grec_entries, bytes;
};
void split_contraction(int64_t tlen, int units, int64_t* chunk, int* nchunk) {
  // aim at about two workgroups per compute unit, chunks of at least 64 and a multiple of 16
  int64_t want = (2 * int64_t(device_cu_count()) + units - 1) / units;
  want = std::max<int64_t>(1, std::min<int64_t>(want, (tlen + 63) / 64));
  int64_t ch = (tlen + want - 1) / want;
  ch = (ch + 15) / 16 * 16;
  *chunk = ch;
  *nchunk = int((tlen + ch - 1) / ch);
}
struct AdaptiveWs {
  float* partial; double* work; float *Cmat, *Sinv, *Rsum; uint16_t* planes; float2 *rec, *grec;
};
AdaptiveWs carve_adaptive(void* ws, const AdaptivePlan& ap, int k, int nb, size_t* bytes) {
  Carver c(ws);
  AdaptiveWs w;
  w.partial = c.take<float>(ap.partial_floats);
  w.work = c.take<double>(size_t(nb) * k * 4 * k);
  w.Cmat = c.take<float>(size_t(nb) * k * k);
  w.Sinv = c.take<float>(size_t(nb) * k * k);
  w.Rsum = c.take<float>(size_t(nb) * k * k);
  w.planes = c.take<uint16_t>(size_t(nb) * kFwdPlanes * k * k);
  w.rec = c.take<float2>(ap.rec_entries);
  w.grec = c.take<float2>(ap.grec_entries);
  if (bytes) *bytes = c.off;
  return w;
}
int plan_adaptive(const cafeq_quant_cfg* cfg, int k, int nb, int rep, int64_t rowsA, int64_t colsA,
                  int64_t rowsB, int64_t colsB, AdaptivePlan* ap) {
  int rc;
  if (!supported_block(k)) return CAFEQ_ERR_UNSUPPORTED;
  if ((rc = resolve_group(cfg, colsA, k, &ap->ga))) return rc;
  if ((rc = resolve_group(cfg, rowsB, k, &ap->gb))) return rc;
  if ((rc = make_plan(k, ap->ga.Gk, rowsA, colsA, &ap->planU, false))) return rc;
  if ((rc = make_plan(k, ap->gb.Gk, colsB, rowsB, &ap->planV, false))) return rc;
  split_contraction(rowsA, nb * (k / 32), &ap->chunkA, &ap->nchunkA);
  split_contraction(colsB, nb * rep * (k / 32), &ap->chunkB, &ap->nchunkB);
  const size_t nz = size_t(std::max(ap->nchunkA, rep * ap->nchunkB));
  ap->partial_floats = size_t(nb) * nz * 2 * k * k;
  // groups that span several segments: records of the requantization's first sweep
  ap->rec_entries = std::max(ap->ga.gspan > 1 ? size_t(colsA / ap->ga.Gk) * size_t(rowsA) : 0,
                             ap->gb.gspan > 1 ? size_t(rowsB / ap->gb.Gk) * size_t(colsB) : 0);
  ap->grec_entries = std::max(ap->ga.gspan > 1 ? size_t(colsA / ap->ga.G) * size_t(rowsA) : 0,
                              ap->gb.gspan > 1 ? size_t(rowsB / ap->gb.G) * size_t(colsB) : 0);
  carve_adaptive(nullptr, *ap, k, nb, &ap->bytes);
  return CAFEQ_OK;
}

void fill_common(CoreParams* p, const cafeq_mat* W, const CorePlan& pl, int rep) {
  p->W = W->data; p->dtype = W->dtype; p->rows = W->rows; p->cols = W->cols; p->ld = W->ld;
  p->rep = rep; p->nseg = pl.nseg; p->nlines = pl.nlines; p->mt_per_seg = pl.mt_per_seg;
  p->n_mt = pl.n_mt; p->nwg = pl.nwg;
  p->Afwd = nullptr; p->Ainv = nullptr;
  p->do_inverse = 0; p->do_grad = 0; p->loss_kind = kLossSur; p->beta = 0.f; p->lse_t = 0.f;
  p->rG = nullptr; p->Zout = nullptr; p->codes = nullptr; p->scales = nullptr;
  p->slot_grad = nullptr; p->slot_hdr = nullptr;
  p->rec = nullptr; p->hdr_ref = nullptr; p->nslot_ref = 0; p->member_ref = nullptr;
  p->fscale = nullptr;
  p->longg = 0; p->gspan = 1; p->grec = nullptr; p->grp = 0;
  p->prep_planes = nullptr; p->prep_lscale = nullptr; p->prep_wsq = nullptr; p->fscale_inv = nullptr;
  p->Tfwd = p->Tback = nullptr; p->rG_out = nullptr;
  p->prep_gtiles = nullptr; p->prep_lines = nullptr;
  p->zkeep = nullptr; p->sweep = 0;
  p->asym = 0; p->mins = nullptr; p->rec_mm = nullptr; p->grec_mm = nullptr;
  p->grid = make_grid(4);
}

// where the loss pass over prepared weights finds them
void set_prepared(CoreParams* p, const cafeq_mat* W, int axis) {
  const bool col = axis == CAFEQ_AXIS_COL;
  const PreparedLayout l = prepared_layout(col ? W->rows : W->cols, col ? W->cols : W->rows, W->dtype, axis);
  const unsigned char* base = static_cast<const unsigned char*>(W->prepared);
  p->prep_wsq = reinterpret_cast<const float*>(base);
  p->prep_lscale = reinterpret_cast<const float*>(base + l.off_lscale);
  p->prep_planes = base + l.off_planes;
  p->prep_lines = col ? nullptr : base + l.off_lines;
}

// Forward sweep(s) of the fused core over one matrix.  `p` holds everything but the group bookkeeping.  For
// groups inside a segment this is one launch.  For groups that span gspan segments: a forward-only sweep that
// records every segment's arg-max, the combination of the records per group, then the sweep proper, which
// takes each group's absmax from the combined records (both sweeps run the same kernel variant, or the second one reads what the
// first one left in zkeep, so they see bit-identical transformed weights).
int run_core(int K, int axis, const GroupPlan& gp, CoreParams p, float2* rec, float2* grec, bool want_rec,
             hipStream_t st, const cafeq_mat* prepared_of = nullptr, float2* rec_mm = nullptr,
             float2* grec_mm = nullptr, float* zkeep = nullptr, bool core32 = false) {
  int rc;
  if (core32) {
    p.rec = want_rec ? rec : nullptr;
    return launch_core32_timed(axis, p, st);
  }
  if (prepared_of) {
    // loss pass over the prepared copy of the weights
    set_prepared(&p, prepared_of, axis);
    p.rec = want_rec ? rec : nullptr;
    return launch_loss_prepared(K, gp.Gk, axis, p, st);
  }
  if (gp.gspan > 1) {
    CoreParams s1 = p;
    s1.do_inverse = 0; s1.do_grad = 0; s1.codes = nullptr; s1.scales = nullptr; s1.Zout = nullptr;
    s1.slot_hdr = zkeep ? p.slot_hdr : nullptr; s1.slot_grad = nullptr;
    s1.zkeep = zkeep; s1.sweep = zkeep ? 1 : 0;
    s1.rec = rec; s1.longg = 1; s1.gspan = 1; s1.grec = nullptr;
    s1.mins = nullptr; s1.rec_mm = p.asym ? rec_mm : nullptr;
    if (p.asym && (!rec_mm || !grec_mm)) return CAFEQ_ERR_INVALID_ARG;
    if ((rc = launch_core(K, gp.Gk, axis, s1, st))) return rc;
    if ((rc = launch_combine_records(rec, gp.gspan, gp.Gk, p.nlines, (p.nseg / gp.gspan), grec, st,
                                     p.asym ? rec_mm : nullptr, p.asym ? grec_mm : nullptr)))
      return rc;
    p.zkeep = zkeep; p.sweep = zkeep ? 2 : 0;
    p.longg = 1; p.gspan = gp.gspan; p.grec = grec; p.rec = nullptr; p.grec_mm = p.asym ? grec_mm : nullptr;
  } else {
    p.rec = want_rec ? rec : nullptr;
  }
  return launch_core(K, gp.Gk, axis, p, st);
}

// Whether the gradient passes of a call can run with one workgroup per (matrix, block) and write the gradient in
// its final form (grad_v2.hip; groups shorter than the block, the others mostly go by records): prepared weights, blocks of 128,
// no row-blocks sharing a transform block, and enough blocks, up to four rounds of workgroups.  Whole evaluations this way against
// partial sums, groups of 64, matrices of 1000 / 2304 / 4608 lines: pairs of 128 blocks in both 81 / 133 / 208 us against 101 / 155 / 219,
// of 64 68 / 100 / 156 against 74 / 109 / 151, of 512 231 / 390 us against 260 / 420: from half of the chip on.  Single matrices,
// whose partial sums are reduced with the losses and the middle factor in one launch: 128 blocks 87 / 141 / 213 us against
// 88 / 141 / 211, 144 blocks 105 / 157 / 240 against 119 / 162 / 247: from nine sixteenths on.
bool grad_owner_eligible(const cafeq_mat* const* mats, const PassPlans* const* pps, int n, int K, int rep) {
  if (K != 128 || rep != 1) return false;
  int64_t jobs = 0;
  for (int i = 0; i < n; ++i) {
    if (!mats[i]->prepared || !pps[i]->two) return false;
    jobs += pps[i]->gpass.nseg;
  }
  const int cus = device_cu_count();
  return jobs <= 4 * int64_t(cus) && jobs * 16 >= int64_t(cus) * (n == 1 ? 9 : 8);
}
GradOwnerJob grad_owner_job(const cafeq_mat* W, int axis, const PassPlans& pp, const MemberWs& m, float* out,
                            int transpose_out) {
  const bool col = axis == CAFEQ_AXIS_COL;
  const PreparedLayout l = prepared_layout(col ? W->rows : W->cols, col ? W->cols : W->rows, W->dtype, axis);
  GradOwnerJob j;
  j.gtiles = static_cast<const unsigned char*>(W->prepared) + l.off_gtiles;
  j.rec = m.grec; j.rG = m.rGreal; j.out = out;
  j.nlines = pp.gpass.nlines; j.nseg = pp.gpass.nseg; j.grp = pp.gp.G; j.transpose_out = transpose_out;
  j.parts = prepared_parts(W->dtype);
  return j;
}

GradGatherJob grad_gather_job(const cafeq_mat* W, int axis, int nb, int rep, const PassPlans& pp, const MemberWs& m, float* out,
                              int transpose_out) {
  GradGatherJob j;
  j.dtype = W->dtype; j.nlines = pp.first.nlines; j.nb = nb; j.rep = rep; j.grp = pp.gp.G; j.transpose_out = transpose_out;
  j.rec = m.grec; j.rG = m.rGreal; j.out = out; j.sorted = m.sorted; j.start = m.start;
  if (axis == CAFEQ_AXIS_COL) {
    j.W = W->data; j.line_stride = W->ld; j.seg_stride = 128;
  } else {
    const PreparedLayout l = prepared_layout(W->cols, W->rows, W->dtype, axis);
    j.W = static_cast<const unsigned char*>(W->prepared) + l.off_lines;
    j.line_stride = 128; j.seg_stride = l.nlp * 128;
  }
  return j;
}

// The gradient pass of the two-pass scheme over one matrix (records in, gradient partials out).
int run_grad_pass(int K, int axis, const cafeq_mat* W, int rep, const PassPlans& pp, const MemberWs& m,
                  int loss_kind, float beta, float lse_t, const float* hdr_ref, int nslot_ref, float* member_ref,
                  CoreParams* pg, hipStream_t st) {
  fill_common(pg, W, pp.gpass, rep);
  pg->loss_kind = loss_kind; pg->beta = beta; pg->lse_t = lse_t;
  pg->rG = m.rGreal; pg->slot_grad = m.slot_grad; pg->rec = m.grec; pg->grp = pp.gp.G;
  pg->hdr_ref = hdr_ref; pg->nslot_ref = nslot_ref; pg->member_ref = member_ref;
  if (W->prepared && K == 128) {
    // the prepared copy also holds the weights in the operand order of this contraction
    const bool col = axis == CAFEQ_AXIS_COL;
    const PreparedLayout l = prepared_layout(col ? W->rows : W->cols, col ? W->cols : W->rows, W->dtype, axis);
    pg->prep_gtiles = static_cast<const unsigned char*>(W->prepared) + l.off_gtiles;
    return launch_grad_v2_timed(*pg, st);
  }
  return launch_grad_pass_timed(K, axis, *pg, st);
}

}  // namespace

namespace cafeq {
namespace {
// Measurement aid: the caller's table of pre-created events (cafeq_set_launch_timing); nothing is created,
// allocated or synchronised here.
cafeq_launch_timing* g_timing = nullptr;
int launch_core_raw(int K, int G, int axis, const CoreParams& p, hipStream_t st) {
  if (p.asym) {
    switch (K) {
      case 32: return launch_core_asym_k32(G, axis, p, st);
      case 64: return launch_core_asym_k64(G, axis, p, st);
      case 128: return launch_core_asym_k128(G, axis, p, st);
      case 256: return launch_core_asym_k256(G, axis, p, st);
      default: return CAFEQ_ERR_UNSUPPORTED;
    }
  }
  switch (K) {
    case 32: return launch_core_k32(G, axis, p, st);
    case 64: return launch_core_k64(G, axis, p, st);
    case 128: return launch_core_k128(G, axis, p, st);
    case 256: return launch_core_k256(G, axis, p, st);
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
}
template <typename F>
int timed_launch(hipStream_t st, F&& launch, int kind = 0) {
  cafeq_launch_timing* t = g_timing;
  if (!t || t->kind != kind || t->count >= t->capacity) return launch();
  const int nth = t->seen++;
  if (t->every > 1 && nth % t->every != 0) return launch();
  const int i = t->count;
  (void)hipEventRecord(static_cast<hipEvent_t>(t->start[i]), st);
  const int rc = launch();
  (void)hipEventRecord(static_cast<hipEvent_t>(t->stop[i]), st);
  t->count = i + 1;
  return rc;
}
}  // namespace
int launch_core(int K, int G, int axis, const CoreParams& p, hipStream_t st) {
  return timed_launch(st, [&] { return launch_core_raw(K, G, axis, p, st); });
}
int launch_core32_timed(int axis, const CoreParams& p, hipStream_t st) {
  return timed_launch(st, [&] { return launch_core32(axis, p, st); });
}
int launch_loss_prepared(int K, int G, int axis, const CoreParams& p, hipStream_t st) {
  return timed_launch(st, [&] { return launch_loss_v2(K, G, axis, p, st); });
}
int launch_loss_prepared_pair(int K, int G, const CoreParams& pa, const CoreParams& pb, hipStream_t st) {
  return timed_launch(st, [&] { return launch_loss_v2_pair(K, G, pa, pb, st); });
}
// the gradient pass over the weights, with the caller's timing events when the table asks for kind 1
int launch_grad_owner_timed(const GradOwnerJob* jobs, int n, int loss_kind, float beta, float lse_t, const double* lse_ms,
                            hipStream_t st, const LossArgs* fold) {
  return timed_launch(st, [&] { return launch_grad_v2_owner(jobs, n, loss_kind, beta, lse_t, lse_ms, st, fold); }, 1);
}
int launch_grad_v2_timed(const CoreParams& p, hipStream_t st) {
  return timed_launch(st, [&] { return launch_grad_v2(p, st); }, 1);
}
int launch_grad_pass_timed(int K, int axis, const CoreParams& p, hipStream_t st) {
  return timed_launch(st, [&] { return launch_grad_pass(K, axis, p, st); }, 1);
}
int launch_grad_gather_timed(int K, const GradGatherJob* jobs, int n, const LossArgs& la, const VArgs* va, hipStream_t st, const RhoGroups* rho) {
  return timed_launch(st, [&] { return launch_grad_gather(K, jobs, n, la, va, st, rho); }, 1);
}
size_t core_lds_bytes(int K, int G, bool do_grad) {
  switch (K) {
    case 32: return core_lds_bytes_k32(G, do_grad);
    case 64: return core_lds_bytes_k64(G, do_grad);
    case 128: return core_lds_bytes_k128(G, do_grad);
    case 256: return core_lds_bytes_k256(G, do_grad);
    default: return 0;
  }
}
}  // namespace cafeq

namespace {
constexpr size_t kLdsLimit = 160 * 1024;
}  // namespace

extern "C" {

const char* cafeq_strerror(int status) {
  switch (status) {
    case CAFEQ_OK: return "ok";
    case CAFEQ_ERR_INVALID_ARG: return "invalid argument";
    case CAFEQ_ERR_BAD_SHAPE: return "shape not divisible as required";
    case CAFEQ_ERR_BAD_ALIGN: return "pointer or leading dimension misaligned";
    case CAFEQ_ERR_UNSUPPORTED: return "configuration not supported by this build";
    case CAFEQ_ERR_SINGULAR: return "singular transform block";
    case CAFEQ_ERR_LAUNCH: return "HIP launch failed";
    case CAFEQ_ERR_WORKSPACE: return "workspace missing or too small";
    default: return "unknown status";
  }
}

int cafeq_pqe(const float* U, const float* V, int64_t rowsA, int64_t colsA, int64_t rowsB, int64_t colsB,
              const cafeq_quant_cfg* cfg, int k, int nb, int rep, const int8_t* codesU, const float* scalesU,
              const int8_t* codesV, const float* scalesV, float* out, void* ws, void* stream) {
  int rc = check_cfg(cfg, false);
  if (rc) return rc;
  if (!U || !V || !codesU || !scalesU || !codesV || !scalesV || !out) return CAFEQ_ERR_INVALID_ARG;
  if (!supported_block(k)) return CAFEQ_ERR_UNSUPPORTED;
  if (nb <= 0 || rep <= 0 || rowsA <= 0 || colsB <= 0) return CAFEQ_ERR_BAD_SHAPE;
  if (colsA != int64_t(nb) * k || rowsB != int64_t(nb) * rep * k || colsB % 4 != 0) return CAFEQ_ERR_BAD_SHAPE;
  if (!aligned16(U) || !aligned16(V) || !aligned16(codesU) || !aligned16(codesV) || !aligned16(scalesU) ||
      !aligned16(scalesV))
    return CAFEQ_ERR_BAD_ALIGN;
  if (!ws) return CAFEQ_ERR_WORKSPACE;
  AdaptivePlan ap;
  if ((rc = plan_adaptive(cfg, k, nb, rep, rowsA, colsA, rowsB, colsB, &ap))) return rc;
  const size_t kk = size_t(k) * k;
  Carver c(ws);
  float* partialU = c.take<float>(size_t(nb) * ap.nchunkA * 3 * kk);
  float* partialV = c.take<float>(size_t(nb) * rep * ap.nchunkB * 3 * kk);
  double* sums = c.take<double>(size_t(nb) * (1 + rep) * 3 * kk + 2 * size_t(nb) * rep);
  return launch_pqe(U, V, rowsA, colsA, rowsB, colsB, k, ap.ga.G, ap.gb.G, nb, rep, codesU, scalesU, codesV, scalesV,
                    ap.chunkA, ap.nchunkA, ap.chunkB, ap.nchunkB, partialU, partialV, sums, out,
                    static_cast<hipStream_t>(stream));
}

int cafeq_version(void) { return 100; }

namespace {
struct OptWs { float* grad; void* orth; void* sub; };
OptWs carve_opt(void* ws, int k, int nb) {
  char* base = static_cast<char*>(ws);
  OptWs w;
  w.grad = reinterpret_cast<float*>(base);
  w.orth = base + align_up(size_t(nb) * k * k * sizeof(float), 256);
  w.sub = static_cast<char*>(w.orth) + orth_ws_any(k, nb);
  return w;
}
// The inverse of iteration s of a learning loop: from scratch first, then warm-started from the previous one.
int loop_inverse(int s, const float* T, int k, int nb, float* Tinv, int* status, void* ws, void* stream) {
  if (s == 0 || small_m(k)) return cafeq_block_inverse(T, k, nb, Tinv, nullptr, nullptr, status, ws, stream);
  return launch_block_inverse_warm(T, k, nb, static_cast<double*>(ws), Tinv, status, static_cast<hipStream_t>(stream));
}
int check_opt(const cafeq_opt_cfg* opt) {
  if (!opt) return CAFEQ_ERR_INVALID_ARG;
  if (opt->steps < 0 || !(opt->lr >= 0.f) || !(opt->lambda_orth >= 0.f)) return CAFEQ_ERR_INVALID_ARG;
  return CAFEQ_OK;
}
}  // namespace

static int dual_impl(const cafeq_mat* A, const cafeq_mat* B, const cafeq_xform* x, const cafeq_quant_cfg* cfg,
                     float lse_t, float* losses, float* gradT, int8_t* codesU, float* scalesU, int8_t* codesV,
                     float* scalesV, void* ws, void* stream, const UpdateHook* hook);

// a loop's step may leave the inverse of the transform it leaves, where its last kernel has that in it (done)
struct LoopInverse { float* Tinv; int* status; bool done; };
static int single_impl(const cafeq_mat* W, const cafeq_xform* x, const cafeq_quant_cfg* cfg, float* losses, float* gradT,
                       int8_t* codes, float* scales, void* ws, void* stream, const UpdateHook* hook, bool loop, LoopInverse* inv = nullptr);

int cafeq_optimize_single(const cafeq_mat* W, float* T, float* Tinv, int k, int nb, int rep,
                          const cafeq_quant_cfg* cfg, const cafeq_opt_cfg* opt, float* history, int* status,
                          void* ws, void* stream) {
  int rc = check_opt(opt);
  if (rc) return rc;
  if (!T || !Tinv || !history) return CAFEQ_ERR_INVALID_ARG;
  if (!ws) return CAFEQ_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const OptWs w = carve_opt(ws, k, nb);
  const int64_t n = int64_t(nb) * k * k;
  cafeq_xform x{T, Tinv, k, nb, rep};
  if ((rc = launch_fill(history, 0.f, int64_t(opt->steps) * 8, st))) return rc;
  // without a regulariser to add in between, the step rides in the epilogue of the gradient's last kernel
  const bool fuse = !(opt->lambda_orth > 0.f) && !small_m(k);
  LoopInverse inv{Tinv, status, false};
  for (int s = 0; s < opt->steps; ++s) {
    float* h = history + size_t(s) * 8;
    if (!inv.done && (rc = loop_inverse(s, T, k, nb, Tinv, status, w.sub, stream))) return rc;
    inv.done = false;
    if (fuse) {
      UpdateHook hook{};
      hook.T = T; hook.lr = opt->lr; hook.denom = opt->normalize ? h + 2 : nullptr;
      // (the last step's inverse is taken from scratch)
      if ((rc = single_impl(W, &x, cfg, h, w.grad, nullptr, nullptr, w.sub, stream, &hook, true, s + 1 < opt->steps ? &inv : nullptr))) return rc;
      continue;
    }
    if ((rc = single_impl(W, &x, cfg, h, w.grad, nullptr, nullptr, w.sub, stream, nullptr, true))) return rc;
    // surrogate / ||W||^2 (history[s][2]) when normalised, then the regulariser's gradient on top
    if (opt->normalize && (rc = launch_div_by_device_scalar(w.grad, h + 2, n, st))) return rc;
    if (opt->lambda_orth > 0.f &&
        (rc = cafeq_orth_penalty(T, k, nb, opt->lambda_orth, h + 4, w.grad, w.orth, stream)))
      return rc;
    if ((rc = cafeq_sgd_update(T, w.grad, opt->lr, nullptr, n, stream))) return rc;
  }
  return cafeq_block_inverse(T, k, nb, Tinv, nullptr, nullptr, status, w.sub, stream);
}

int cafeq_optimize_pair(const cafeq_mat* A, const cafeq_mat* B, float* T, float* Tinv, int k, int nb, int rep,
                        const cafeq_quant_cfg* cfg, float lse_t, const cafeq_opt_cfg* opt, float* moments,
                        float* history, int* status, void* ws, void* stream) {
  int rc = check_opt(opt);
  if (rc) return rc;
  if (!T || !Tinv || !history || !moments) return CAFEQ_ERR_INVALID_ARG;
  if (!ws) return CAFEQ_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const OptWs w = carve_opt(ws, k, nb);
  const int64_t n = int64_t(nb) * k * k;
  cafeq_xform x{T, Tinv, k, nb, rep};
  if ((rc = launch_fill(history, 0.f, int64_t(opt->steps) * 8, st))) return rc;
  if ((rc = launch_fill(moments, 0.f, 2 * n, st))) return rc;
  const bool fuse_adam = !(opt->lambda_orth > 0.f) && !small_m(k);
  for (int s = 0; s < opt->steps; ++s) {
    float* h = history + size_t(s) * 8;
    if ((rc = loop_inverse(s, T, k, nb, Tinv, status, w.sub, stream))) return rc;
    if (fuse_adam) {
      // the Adam step rides in the epilogue of the gradient's last kernel (no regulariser to add in between)
      if (!(opt->beta1 >= 0.0 && opt->beta1 < 1.0 && opt->beta2 >= 0.0 && opt->beta2 < 1.0)) return CAFEQ_ERR_INVALID_ARG;
      UpdateHook hook{};
      hook.T = T; hook.m = moments; hook.v = moments + n;
      hook.lr = float(opt->lr); hook.beta1 = float(opt->beta1); hook.omb1 = float(1.0 - opt->beta1);
      hook.beta2 = float(opt->beta2); hook.omb2 = float(1.0 - opt->beta2); hook.eps = float(opt->eps);
      hook.c1 = float(1.0 / (1.0 - pow(opt->beta1, double(s + 1))));
      hook.c2 = float(1.0 / (1.0 - pow(opt->beta2, double(s + 1))));
      if ((rc = dual_impl(A, B, &x, cfg, lse_t, h, w.grad, nullptr, nullptr, nullptr, nullptr, w.sub, stream, &hook)))
        return rc;
      continue;
    }
    if ((rc = cafeq_dual_proxy_loss_fwd_bwd(A, B, &x, cfg, lse_t, h, w.grad, nullptr, nullptr, nullptr, nullptr, w.sub,
                                            stream)))
      return rc;
    if (opt->lambda_orth > 0.f &&
        (rc = cafeq_orth_penalty(T, k, nb, opt->lambda_orth, h + 6, w.grad, w.orth, stream)))
      return rc;
    if ((rc = cafeq_adam_update(T, w.grad, moments, moments + n, s + 1, opt->lr, opt->beta1, opt->beta2, opt->eps, n,
                                stream)))
      return rc;
  }
  return cafeq_block_inverse(T, k, nb, Tinv, nullptr, nullptr, status, w.sub, stream);
}


namespace cafeq {
namespace {
__global__ __launch_bounds__(256) void stream_read_kernel(const uintx4* __restrict__ p, size_t n16, unsigned* sink) {
  unsigned acc = 0;
  const size_t stride = size_t(gridDim.x) * 1024;
  size_t base = size_t(blockIdx.x) * 1024 + threadIdx.x;
  for (; base + 768 < n16; base += stride) {
    uintx4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(p + base + 256 * u);
#pragma unroll
    for (int u = 0; u < 4; ++u) acc ^= v[u][0] ^ v[u][1] ^ v[u][2] ^ v[u][3];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {       // the last, partial step of 1024 vectors (every later step lies beyond the end)
    const size_t i = base + 256 * u;
    if (i < n16) {
      const uintx4 v = p[i];
      acc ^= v[0] ^ v[1] ^ v[2] ^ v[3];
    }
  }
  if (acc == 0x5EEDF00Du) sink[0] = acc;
}
}  // namespace
}  // namespace cafeq

int cafeq_stream_read_probe(const void* buf, size_t bytes, void* sink, void* stream) {
  if (!buf || !sink || bytes < 16 || bytes % 16 != 0 || reinterpret_cast<uintptr_t>(buf) % 16 != 0) return CAFEQ_ERR_INVALID_ARG;
  const size_t n16 = bytes / 16;
  const size_t steps = (n16 + 1023) / 1024;
  const unsigned grid = unsigned(std::min<size_t>(steps, 8192));
  hipLaunchKernelGGL(cafeq::stream_read_kernel, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<const cafeq::uintx4*>(buf), n16, static_cast<unsigned*>(sink));
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}

int cafeq_set_launch_timing(cafeq_launch_timing* t) {
  if (t && (t->capacity < 0 || t->count < 0 || (t->capacity > 0 && (!t->start || !t->stop)))) return CAFEQ_ERR_INVALID_ARG;
  cafeq::g_timing = t;
  return CAFEQ_OK;
}

size_t cafeq_workspace_bytes(int call_id, const cafeq_mat* a, const cafeq_mat* b, const cafeq_xform* x,
                             const cafeq_quant_cfg* cfg) {
  if (x && small_m(x->k) && call_id != CAFEQ_CALL_ORTH_PENALTY && call_id != CAFEQ_CALL_OPTIMIZE_SINGLE &&
      call_id != CAFEQ_CALL_OPTIMIZE_PAIR) {
    // blocks smaller than 32: the embedding's scratch in front of what the same call needs with blocks of 32
    int64_t nb32 = 0;
    switch (call_id) {
      case CAFEQ_CALL_PROXY_LOSS:
        if (!a || !cfg) return 0;
        nb32 = small_nb32(x, cfg->axis == CAFEQ_AXIS_COL ? a->cols : a->rows);
        break;
      case CAFEQ_CALL_DUAL_PROXY_LOSS:
        if (!a || x->rep != 1) return 0;
        nb32 = small_nb32(x, a->cols);
        break;
      case CAFEQ_CALL_APPLY_TRANSFORM:
      case CAFEQ_CALL_BLOCK_INVERSE:
        nb32 = (int64_t(x->nb) * (x->rep > 0 ? x->rep : 1) * x->k) / 32;
        if (nb32 * 32 != int64_t(x->nb) * (x->rep > 0 ? x->rep : 1) * x->k) nb32 = 0;
        break;
      default: return 0;   // Alg. 1 and the paired error work per head: blocks of 32 and more
    }
    if (nb32 <= 0 || nb32 > (int64_t(1) << 30)) return 0;
    const cafeq_xform x32{nullptr, nullptr, 32, int(nb32), 1};
    const size_t sub = cafeq_workspace_bytes(call_id, a, b, &x32, cfg);
    return sub ? carve_small(nullptr, nb32).head + sub : 0;
  }
  switch (call_id) {
    case CAFEQ_CALL_RTN_QUANTIZE:
      if (!a) return 0;
      return align_up(rtn_partials_capacity(a->rows, a->cols) * sizeof(double), 256);
    case CAFEQ_CALL_APPLY_TRANSFORM:
      if (!x) return 0;
      return align_up(size_t(x->nb) * kFwdPlanes * x->k * x->k * sizeof(uint16_t), 256);
    case CAFEQ_CALL_BLOCK_INVERSE:
      if (!x) return 0;
      if (x->k == 256) return align_up(inverse256_workspace_bytes(x->nb), 256);
      return align_up(size_t(x->nb) * x->k * 2 * x->k * sizeof(double), 256);
    case CAFEQ_CALL_PROXY_LOSS: {
      if (!a || !x || !cfg) return 0;
      const bool col = cfg->axis == CAFEQ_AXIS_COL;
      const int64_t naxis = col ? a->cols : a->rows, nlines = col ? a->rows : a->cols;
      GroupPlan gp;
      if (resolve_group(cfg, naxis, x->k, &gp)) return 0;
      PassPlans pg, pn;
      const bool mm = is_minmax(cfg);
      if (plan_passes(x->k, gp, nlines, naxis, false, &pn, false, mm)) return 0;
      size_t bytes = carve_single(nullptr, pn, x->nb, false).bytes;
      // (where the gradient has no kernel the forward-only size is still reported)
      if (!plan_passes(x->k, gp, nlines, naxis, true, &pg, false, mm)) bytes = std::max(bytes, carve_single(nullptr, pg, x->nb, true).bytes);
      if (gather_possible(x->k, gp, true) && !plan_passes(x->k, gp, nlines, naxis, true, &pg, false, mm, 1, true))
        bytes = std::max(bytes, carve_single(nullptr, pg, x->nb, true).bytes);
      return bytes;
    }
    case CAFEQ_CALL_DUAL_PROXY_LOSS: {
      if (!a || !b || !x || !cfg) return 0;
      GroupPlan ga, gb;
      if (resolve_group(cfg, a->cols, x->k, &ga) || resolve_group(cfg, b->rows, x->k, &gb)) return 0;
      PassPlans qa, qb, na, nbp;
      const bool mm = is_minmax(cfg);
      if (plan_passes(x->k, ga, a->rows, a->cols, false, &na, false, mm) ||
          plan_passes(x->k, gb, b->cols, b->rows, false, &nbp, false, mm))
        return 0;
      size_t bytes = carve_dual(nullptr, na, nbp, x->nb, false).bytes;
      if (!plan_passes(x->k, ga, a->rows, a->cols, true, &qa, false, mm) &&
          !plan_passes(x->k, gb, b->cols, b->rows, true, &qb, false, mm))
        bytes = std::max(bytes, carve_dual(nullptr, qa, qb, x->nb, true).bytes);
      if (gather_possible(x->k, ga, true) && gather_possible(x->k, gb, true) &&
          !plan_passes(x->k, ga, a->rows, a->cols, true, &qa, false, mm, 1, true) &&
          !plan_passes(x->k, gb, b->cols, b->rows, true, &qb, false, mm, 1, true))
        bytes = std::max(bytes, carve_dual(nullptr, qa, qb, x->nb, true).bytes);
      return bytes;
    }
    case CAFEQ_CALL_ORTH_PENALTY:
      if (!x) return 0;
      return orth_ws_any(x->k, x->nb);
    case CAFEQ_CALL_OPTIMIZE_SINGLE:
    case CAFEQ_CALL_OPTIMIZE_PAIR: {
      // gradient buffer + regulariser scratch + the larger of the sub-calls' workspaces
      if (!x) return 0;
      const size_t sub = std::max(
          cafeq_workspace_bytes(call_id == CAFEQ_CALL_OPTIMIZE_SINGLE ? CAFEQ_CALL_PROXY_LOSS : CAFEQ_CALL_DUAL_PROXY_LOSS,
                                a, b, x, cfg),
          cafeq_workspace_bytes(CAFEQ_CALL_BLOCK_INVERSE, a, b, x, cfg));
      if (sub == 0) return 0;
      return align_up(size_t(x->nb) * x->k * x->k * sizeof(float), 256) + orth_ws_any(x->k, x->nb) + sub;
    }
    case CAFEQ_CALL_PQE: {
      if (!a || !b || !x || !cfg) return 0;
      AdaptivePlan ap;
      if (plan_adaptive(cfg, x->k, x->nb, x->rep, a->rows, a->cols, b->rows, b->cols, &ap)) return 0;
      const size_t kk = size_t(x->k) * x->k;
      Carver c(nullptr);
      c.take<float>(size_t(x->nb) * ap.nchunkA * 3 * kk);
      c.take<float>(size_t(x->nb) * x->rep * ap.nchunkB * 3 * kk);
      c.take<double>(size_t(x->nb) * (1 + x->rep) * 3 * kk + 2 * size_t(x->nb) * x->rep);
      return c.off;
    }
    case CAFEQ_CALL_ADAPTIVE_ROUND: {
      // a: U [rowsA][nb*k], b: V [nb*rep*k][colsB]
      if (!a || !b || !x || !cfg) return 0;
      AdaptivePlan ap;
      if (plan_adaptive(cfg, x->k, x->nb, x->rep, a->rows, a->cols, b->rows, b->cols, &ap)) return 0;
      return ap.bytes;
    }
    default:
      return 0;
  }
}

size_t cafeq_prepared_bytes(const cafeq_mat* W, int axis) {
  if (!W || W->rows <= 0 || W->cols <= 0 || (axis != CAFEQ_AXIS_COL && axis != CAFEQ_AXIS_ROW)) return 0;
  const bool col = axis == CAFEQ_AXIS_COL;
  const int64_t nlines = col ? W->rows : W->cols, naxis = col ? W->cols : W->rows;
  if (naxis % 128 != 0) return 0;
  return prepared_layout(nlines, naxis, W->dtype, axis).bytes;
}

int cafeq_prepare_weights(const cafeq_mat* W, int axis, void* prepared, void* stream) {
  int rc = check_mat(W);
  if (rc) return rc;
  if (axis != CAFEQ_AXIS_COL && axis != CAFEQ_AXIS_ROW) return CAFEQ_ERR_INVALID_ARG;
  if (!prepared) return CAFEQ_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(prepared) & 255u) != 0) return CAFEQ_ERR_BAD_ALIGN;
  return launch_prepare(W, axis, prepared, static_cast<hipStream_t>(stream));
}

int cafeq_rtn_quantize(const cafeq_mat* W, const cafeq_quant_cfg* cfg, int8_t* codes, float* scales,
                       float* err_sq, void* ws, void* stream) {
  int rc = check_mat(W);
  if (rc) return rc;
  rc = check_cfg(cfg, true);
  if (rc) return rc;
  if (!codes) return CAFEQ_ERR_INVALID_ARG;
  if (!aligned16(codes) || (scales && !aligned16(scales))) return CAFEQ_ERR_BAD_ALIGN;
  const int64_t line = cfg->axis == CAFEQ_AXIS_COL ? W->cols : W->rows;
  const int64_t g = cfg->group == 0 ? line : cfg->group;
  if (line % g != 0) return CAFEQ_ERR_BAD_SHAPE;
  if (err_sq && !ws) return CAFEQ_ERR_WORKSPACE;
  RtnArgs a;
  a.W = W->data; a.dtype = W->dtype; a.rows = W->rows; a.cols = W->cols; a.ld = W->ld;
  a.axis = cfg->axis; a.group = cfg->group; a.grid = make_grid(cfg->bits);
  a.codes = codes; a.scales = scales; a.mins = nullptr;
  a.partial = err_sq ? static_cast<double*>(ws) : nullptr;
  a.err_sq = err_sq;
  return launch_rtn(a, static_cast<hipStream_t>(stream));
}

int cafeq_rtn_quantize_minmax(const cafeq_mat* W, const cafeq_quant_cfg* cfg, uint8_t* codes, float* scales,
                              float* mins, float* err_sq, void* ws, void* stream) {
  int rc = check_mat(W);
  if (rc) return rc;
  if (!cfg || cfg->bits < 1 || cfg->bits > 8 || cfg->group < 0) return CAFEQ_ERR_INVALID_ARG;
  if (cfg->axis != CAFEQ_AXIS_COL && cfg->axis != CAFEQ_AXIS_ROW) return CAFEQ_ERR_INVALID_ARG;
  if (!codes) return CAFEQ_ERR_INVALID_ARG;
  if (!aligned16(codes) || (scales && !aligned16(scales)) || (mins && !aligned16(mins))) return CAFEQ_ERR_BAD_ALIGN;
  const int64_t line = cfg->axis == CAFEQ_AXIS_COL ? W->cols : W->rows;
  const int64_t g = cfg->group == 0 ? line : cfg->group;
  if (line % g != 0) return CAFEQ_ERR_BAD_SHAPE;
  if (err_sq && !ws) return CAFEQ_ERR_WORKSPACE;
  RtnArgs a;
  a.W = W->data; a.dtype = W->dtype; a.rows = W->rows; a.cols = W->cols; a.ld = W->ld;
  a.axis = cfg->axis; a.group = cfg->group; a.grid = make_grid(2);
  a.codes = reinterpret_cast<int8_t*>(codes); a.scales = scales; a.mins = mins;
  a.partial = err_sq ? static_cast<double*>(ws) : nullptr;
  a.err_sq = err_sq;
  return launch_rtn_minmax(a, cfg->bits, static_cast<hipStream_t>(stream));
}

int cafeq_block_inverse(const float* T, int k, int nb, float* Tinv, float* rho_row, float* rho_col,
                        int* status, void* ws, void* stream) {
  if (!T || !Tinv) return CAFEQ_ERR_INVALID_ARG;
  if (nb < 1) return CAFEQ_ERR_BAD_SHAPE;
  if (const int m = small_m(k)) {
    // a run of 32 / k blocks as one block-diagonal block of 32 (its inverse is block-diagonal too; the squared
    // row / column norms keep their positions; a singular block marks its whole run)
    if (nb % m != 0) return CAFEQ_ERR_BAD_SHAPE;
    if (!ws) return CAFEQ_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int nb32 = nb / m;
    const SmallWs w = carve_small(ws, nb32);
    int rc;
    if ((rc = launch_embed_blocks(T, k, nb, 1, nb32, w.T32, st))) return rc;
    if ((rc = cafeq_block_inverse(w.T32, 32, nb32, w.P32, rho_row, rho_col, status ? w.st32 : nullptr, w.sub, stream)))
      return rc;
    if ((rc = launch_gather_blocks(w.P32, k, nb, 1, Tinv, st))) return rc;
    if (status && (rc = launch_expand_status(w.st32, m, nb, status, st))) return rc;
    return CAFEQ_OK;
  }
  if (k != 32 && k != 64 && k != 128 && k != 256) return CAFEQ_ERR_UNSUPPORTED;
  if (!ws) return CAFEQ_ERR_WORKSPACE;
  return launch_block_inverse(T, k, nb, static_cast<double*>(ws), Tinv, rho_row, rho_col, status,
                              static_cast<hipStream_t>(stream));
}

int cafeq_apply_transform(const cafeq_mat* W, const cafeq_xform* x, int axis, int side, float* Z,
                          void* ws, void* stream) {
  int rc = check_mat(W);
  if (rc) return rc;
  if (side != CAFEQ_SIDE_T && side != CAFEQ_SIDE_TINV) return CAFEQ_ERR_INVALID_ARG;
  if (x && small_m(x->k)) {
    if ((rc = check_small_xform(x, side == CAFEQ_SIDE_TINV))) return rc;
    if ((rc = check_axis_len(W, x, axis))) return rc;
    if (!ws) return CAFEQ_ERR_WORKSPACE;
    const int64_t nb32 = small_nb32(x, axis == CAFEQ_AXIS_COL ? W->cols : W->rows);
    if (nb32 <= 0) return CAFEQ_ERR_BAD_SHAPE;
    const SmallWs w = carve_small(ws, nb32);
    if ((rc = launch_embed_blocks(side == CAFEQ_SIDE_T ? x->T : x->Tinv, x->k, x->nb, x->rep, int(nb32), w.T32,
                                  static_cast<hipStream_t>(stream))))
      return rc;
    const cafeq_xform x32{w.T32, w.T32, 32, int(nb32), 1};
    return cafeq_apply_transform(W, &x32, axis, side, Z, w.sub, stream);
  }
  rc = check_xform(x, side == CAFEQ_SIDE_TINV);
  if (rc) return rc;
  rc = check_axis_len(W, x, axis);
  if (rc) return rc;
  if (!Z) return CAFEQ_ERR_INVALID_ARG;
  if (!aligned16(Z)) return CAFEQ_ERR_BAD_ALIGN;
  if (!ws) return CAFEQ_ERR_WORKSPACE;
  const bool col = axis == CAFEQ_AXIS_COL;
  CorePlan pl;
  rc = make_plan(x->k, x->k, col ? W->rows : W->cols, col ? W->cols : W->rows, &pl, false);
  if (rc) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  uint16_t* planes = static_cast<uint16_t*>(ws);
  // half-precision forward operands where the kernel variant exists: two planes, and the per-block factors
  // in the room of the third
  float* fs = core_forward_f16(x->k, x->k, 4) ? reinterpret_cast<float*>(planes + size_t(x->nb) * 2 * x->k * x->k) : nullptr;
  {
    const SplitRequest req{side == CAFEQ_SIDE_T ? x->T : x->Tinv, planes, col ? 1 : 0, fs ? 2 : kFwdPlanes, fs};
    if ((rc = launch_split_planes_multi(&req, 1, x->k, x->nb, st))) return rc;
  }
  CoreParams p;
  fill_common(&p, W, pl, x->rep);
  p.Afwd = planes; p.Ainv = nullptr; p.fscale = fs;
  p.Zout = Z;
  return launch_core(x->k, x->k, axis, p, st);
}

// hook (learning loop only; blocks of 32 and more): the last kernel of the gradient applies the gradient-descent step
// to T instead of storing the gradient (gradT is then scratch).  loop: called from a learning loop, with a hook or without.
static int single_impl(const cafeq_mat* W, const cafeq_xform* x, const cafeq_quant_cfg* cfg, float* losses, float* gradT,
                       int8_t* codes, float* scales, void* ws, void* stream, const UpdateHook* hook, bool loop, LoopInverse* inv) {
  int rc = check_mat(W);
  if (rc) return rc;
  rc = check_cfg(cfg, true, true);
  if (rc) return rc;
  if (x && small_m(x->k)) {
    if (hook) return CAFEQ_ERR_INVALID_ARG;
    if ((rc = check_small_xform(x, true))) return rc;
    if ((rc = check_axis_len(W, x, cfg->axis))) return rc;
    if (!ws) return CAFEQ_ERR_WORKSPACE;
    if (gradT && !aligned16(gradT)) return CAFEQ_ERR_BAD_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t nb32 = small_nb32(x, cfg->axis == CAFEQ_AXIS_COL ? W->cols : W->rows);
    if (nb32 <= 0) return CAFEQ_ERR_BAD_SHAPE;
    const SmallWs w = carve_small(ws, nb32);
    if ((rc = launch_embed_blocks(x->T, x->k, x->nb, x->rep, int(nb32), w.T32, st))) return rc;
    if ((rc = launch_embed_blocks(x->Tinv, x->k, x->nb, x->rep, int(nb32), w.P32, st))) return rc;
    const cafeq_xform x32{w.T32, w.P32, 32, int(nb32), 1};
    if ((rc = single_impl(W, &x32, cfg, losses, gradT ? w.G32 : nullptr, codes, scales, w.sub, stream, nullptr, loop))) return rc;
    return gradT ? launch_gather_blocks(w.G32, x->k, x->nb, x->rep, gradT, st) : CAFEQ_OK;
  }
  rc = check_xform(x, true);
  if (rc) return rc;
  rc = check_axis_len(W, x, cfg->axis);
  if (rc) return rc;
  if (!losses) return CAFEQ_ERR_INVALID_ARG;
  if (!ws) return CAFEQ_ERR_WORKSPACE;
  if ((codes && !aligned16(codes)) || (scales && !aligned16(scales)) || (gradT && !aligned16(gradT)))
    return CAFEQ_ERR_BAD_ALIGN;
  const bool col = cfg->axis == CAFEQ_AXIS_COL;
  const int64_t naxis = col ? W->cols : W->rows, nlines = col ? W->rows : W->cols;
  const int K = x->k, nb = x->nb;
  GroupPlan gp;
  rc = resolve_group(cfg, naxis, K, &gp);
  if (rc) return rc;
  const bool grad = gradT != nullptr;
  const bool asym = is_minmax(cfg);
  // Gradient descent at two bits takes steps nine times those at three and amplifies what rounds: of 60 loops of eight steps 22
  // end more than 1e-5 (and up to 1) elsewhere by records than by the product, 10 where the weights move by half a unit in
  // their last place, although the gradient itself is ten times closer to float64's.  These loops, with or without a regulariser and
  // whatever the block, take their sums over the lines from the product (blocks of 32 and 64 also on the loss pass' way), so that where one ends
  // does not turn on the sizes from which records are the faster way.  It does turn on every other rounding of an iteration (the
  // gradient's third part at k = 32 with groups of 32, the chain through the inverse at k = 128).  Evaluations do not depend on the bits.
  bool v2 = v2_eligible(W, K, gp, cfg, !col && (codes || scales)) && v2_pays(W, K, gp, nlines, naxis, codes || scales, !col);
  const bool gather = gather_possible(K, gp, has_lines(W, cfg->axis)) && gather_pays(W, K, gp, nlines, naxis, asym, false, v2, !col) &&
                      !(loop && cfg->bits == 2);
  if (K < 128 && grad && !gather) v2 = false;   // (the loss pass forms the gradient on its way)
  PassPlans pp;
  rc = plan_passes(K, gp, nlines, naxis, grad, &pp, v2, asym, 1, gather);
  if (rc) return rc;
  const CorePlan& pl = pp.first;
  {
    const size_t lds = core_lds_bytes(K, gp.Gk, pp.fused);
    if (lds == 0 || lds > kLdsLimit) return CAFEQ_ERR_UNSUPPORTED;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  SingleWs w = carve_single(ws, pp, nb, grad);
  const QGrid grid = grid_for(cfg);
  const float beta = beta_for(cfg, grid);
  const bool f16 = v2 || core_forward_f16(K, gp.Gk, cfg->bits);

  CoreParams p;
  fill_common(&p, W, pl, x->rep);
  // forward operand [out][in]: T^T (COL) or T (ROW); inverse operand: Tinv^T or Tinv
  // (a pass that splits them itself: no planes, and it writes every header and rG)
  if (!pp.core32 && !(v2 && v2_splits_planes(K, false, codes || scales))) {
    // (prepared weights: float16 planes for both operands, scaled so that the rounding error fits float16)
    const SplitRequest req[2] = {{x->T, w.m.pfwd, col ? 1 : 0, v2 ? v2_fwd_parts(K) : f16 ? 2 : kFwdPlanes, f16 ? w.m.fs : nullptr, v2 ? 1 : 0, v2 ? 4 : 14},
                                 {x->Tinv, w.m.pinv, col ? 1 : 0, kInvPlanes, v2 ? w.m.fsi : nullptr, 0, 4}};
    // rho per axis index, its sums per segment-level group (the loss sweep) and per group (the gradient pass)
    // (groups inside a block, or of a few whole blocks: the same launch)
    const bool rg_inline = rho_groups_inline(K, nb, gp.Gk, x->rep);
    const RhoRequest rho{x->Tinv, w.rho, col ? 1 : 0, rg_inline ? w.m.rG : nullptr, gp.Gk, x->rep};
    if ((rc = launch_split_planes_multi(req, 2, K, nb, st, w.slot_hdr, pl.nslot, &rho, 1))) return rc;
    if (!rg_inline && (rc = launch_rho_groups(w.rho, K, x->rep, gp.Gk, naxis / gp.Gk, w.m.rG, st))) return rc;
    // (by records the launch that sorts them takes these sums along)
    if (grad && !gather && gp.gspan > 1 && (rc = launch_rho_groups(w.rho, K, x->rep, gp.G, naxis / gp.G, w.m.rGreal, st))) return rc;
  }
  p.Afwd = w.m.pfwd; p.Ainv = w.m.pinv; p.fscale = f16 ? w.m.fs : nullptr; p.fscale_inv = v2 ? w.m.fsi : nullptr;
  p.grid = grid; p.do_inverse = 1; p.do_grad = pp.fused ? 1 : 0; p.loss_kind = kLossSur; p.beta = beta;
  p.Tfwd = x->T; p.Tback = x->Tinv; p.rG_out = w.m.rG;
  p.rG = w.m.rG; p.codes = codes; p.scales = scales; p.slot_grad = w.m.slot_grad; p.slot_hdr = w.slot_hdr;
  p.asym = asym ? 1 : 0;
  p.mins = asym && scales ? scales + nlines * (naxis / gp.G) : nullptr;   // the minima follow the scales
  if ((rc = run_core(K, cfg->axis, gp, p, w.m.rec, w.m.grec, pp.two, st, v2 ? W : nullptr, w.m.rec_mm, w.m.grec_mm, w.m.zkeep, pp.core32)))
    return rc;
  const cafeq_mat* mats[1] = {W};
  const PassPlans* pps[1] = {&pp};
  const bool owner = grad && !pp.gather && grad_owner_eligible(mats, pps, 1, K, x->rep);
  // (with one workgroup per block in the gradient pass, its first workgroup reduces the losses: one launch less)
  // (with gradient partials, the loss reduction rides in the launch that reduces them)
  if (!grad && (rc = launch_reduce_losses(kLossSur, w.slot_hdr, int(pl.nslot), nullptr, 0, beta, 0.f, 0, losses,
                                          w.lse_ms, st)))
    return rc;
  if (grad) {
    // path through Z (fused into the pass above, or a second pass over the weights from its
    // arg-max records), then the path through rho(P): -2 P^T Mmid P^T
    CoreParams pg = p;
    if (pp.gather) {
      // (with the middle factor of the rho path and the loss reduction)
      const GradGatherJob job = grad_gather_job(W, cfg->axis, nb, x->rep, pp, w.m, gradT, col ? 1 : 0);
      const VArgs va = mmid_args(p, K, pl.L, gp.Gk, x->Tinv, col ? 1 : 0, w.mmid);
      LossArgs la{};
      la.hdrA = w.slot_hdr; la.nslotA = int(pl.nslot); la.kind = kLossSur; la.beta = beta; la.losses = losses;
      la.lse_ms = w.lse_ms;
      const RhoGroups rho{w.rho, w.m.rGreal, 31 - __builtin_clz(unsigned(K)), x->rep, gp.G, unsigned(naxis / gp.G)};
      if ((rc = launch_grad_gather_timed(K, &job, 1, la, &va, st, gp.gspan > 1 ? &rho : nullptr))) return rc;
    } else if (owner) {
      const GradOwnerJob job = grad_owner_job(W, cfg->axis, pp, w.m, gradT, col ? 1 : 0);
      LossArgs la{};
      la.hdrA = w.slot_hdr; la.nslotA = int(pl.nslot); la.kind = kLossSur; la.beta = beta; la.losses = losses;
      la.lse_ms = w.lse_ms;
      if ((rc = launch_grad_owner_timed(&job, 1, kLossSur, beta, 0.f, nullptr, st, &la))) return rc;
    } else {
      if (pp.two &&
          (rc = run_grad_pass(K, cfg->axis, W, x->rep, pp, w.m, kLossSur, beta, 0.f, nullptr, 0, nullptr, &pg, st)))
        return rc;
      if (K == 32) {
        if (inv) inv->done = true;
        return launch_tail_chain32(pg, p, gp.Gk, pp.fused, nb, col ? 1 : 0, gradT, x->Tinv, col ? 1 : 0, beta, int(pl.nslot), losses, w.lse_ms,
                                   st, hook, inv ? inv->Tinv : nullptr, inv ? inv->status : nullptr);
      }
      // gradient reduction, the middle factor of the rho path and the loss reduction in one launch
      if ((rc = launch_single_tail(pg, p, K, gp.Gk, pp.fused, nb, col ? 1 : 0, gradT, x->Tinv, col ? 1 : 0, w.mmid, beta,
                                   int(pl.nslot), losses, w.lse_ms, st)))
        return rc;
    }
    if (owner && (rc = launch_build_mmid(p, K, gp.Gk, nb, x->Tinv, col ? 1 : 0, w.mmid, st))) return rc;
    if ((rc = launch_bgemm_chain(x->Tinv, w.mmid, w.x1, gradT, K, nb, -2.f, 1.f, st, hook))) return rc;
  }
  return CAFEQ_OK;
}

int cafeq_proxy_loss_fwd_bwd(const cafeq_mat* W, const cafeq_xform* x, const cafeq_quant_cfg* cfg,
                             float* losses, float* gradT, int8_t* codes, float* scales, void* ws,
                             void* stream) {
  return single_impl(W, x, cfg, losses, gradT, codes, scales, ws, stream, nullptr, false);
}

// hook (learning loop only; blocks of 32 and more): the last kernel of the gradient applies the Adam step to T, m
// and v instead of storing the gradient (gradT is then scratch)
static int dual_impl(const cafeq_mat* A, const cafeq_mat* B, const cafeq_xform* x, const cafeq_quant_cfg* cfg,
                     float lse_t, float* losses, float* gradT, int8_t* codesU, float* scalesU, int8_t* codesV,
                     float* scalesV, void* ws, void* stream, const UpdateHook* hook) {
  int rc = check_mat(A);
  if (rc) return rc;
  rc = check_mat(B);
  if (rc) return rc;
  rc = check_cfg(cfg, false, true);
  if (rc) return rc;
  if (x && small_m(x->k)) {
    // (row-blocks that share a small block do not line up with blocks of 32: rep must be 1 here)
    if (hook) return CAFEQ_ERR_INVALID_ARG;
    if ((rc = check_small_xform(x, true))) return rc;
    if (x->rep != 1) return CAFEQ_ERR_UNSUPPORTED;
    if (A->cols != int64_t(x->nb) * x->k || B->rows != A->cols) return CAFEQ_ERR_BAD_SHAPE;
    if (!ws) return CAFEQ_ERR_WORKSPACE;
    if (gradT && !aligned16(gradT)) return CAFEQ_ERR_BAD_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t nb32 = small_nb32(x, A->cols);
    if (nb32 <= 0) return CAFEQ_ERR_BAD_SHAPE;
    const SmallWs w = carve_small(ws, nb32);
    if ((rc = launch_embed_blocks(x->T, x->k, x->nb, 1, int(nb32), w.T32, st))) return rc;
    if ((rc = launch_embed_blocks(x->Tinv, x->k, x->nb, 1, int(nb32), w.P32, st))) return rc;
    const cafeq_xform x32{w.T32, w.P32, 32, int(nb32), 1};
    if ((rc = cafeq_dual_proxy_loss_fwd_bwd(A, B, &x32, cfg, lse_t, losses, gradT ? w.G32 : nullptr, codesU, scalesU,
                                            codesV, scalesV, w.sub, stream)))
      return rc;
    return gradT ? launch_gather_blocks(w.G32, x->k, x->nb, 1, gradT, st) : CAFEQ_OK;
  }
  rc = check_xform(x, true);
  if (rc) return rc;
  if (!losses) return CAFEQ_ERR_INVALID_ARG;
  if (!(lse_t > 0.f)) return CAFEQ_ERR_INVALID_ARG;
  if (!ws) return CAFEQ_ERR_WORKSPACE;
  const int K = x->k, nb = x->nb;
  if (A->cols != int64_t(nb) * K || B->rows != int64_t(nb) * x->rep * K) return CAFEQ_ERR_BAD_SHAPE;
  GroupPlan ga, gb;
  if ((rc = resolve_group(cfg, A->cols, K, &ga))) return rc;
  if ((rc = resolve_group(cfg, B->rows, K, &gb))) return rc;
  const bool grad = gradT != nullptr;
  const bool asym = is_minmax(cfg);
  const bool gather = gather_possible(K, ga, has_lines(A, CAFEQ_AXIS_COL)) && gather_possible(K, gb, has_lines(B, CAFEQ_AXIS_ROW)) &&
                      gather_pays(A, K, ga, A->rows, A->cols, asym, true, false, false) &&
                      gather_pays(B, K, gb, B->cols, B->rows, asym, true, false, true);
  bool v2A = v2_eligible(A, K, ga, cfg, false), v2B = v2_eligible(B, K, gb, cfg, codesV || scalesV);
  // both loss passes over prepared weights in one launch, each member on half of the chip: when neither writes
  // codes or scales and both use the same group length
  bool pair_launch = v2A && v2B && !codesU && !scalesU && !codesV && !scalesV && ga.Gk == gb.Gk;
  if (pair_launch) {
    v2A = v2B = pair_launch = v2_pair_pays(A, B, K, ga);
  } else {
    v2A = v2A && v2_pays(A, K, ga, A->rows, A->cols, codesU || scalesU, false);
    v2B = v2B && v2_pays(B, K, gb, B->cols, B->rows, codesV || scalesV, true);
  }
  if (K < 128 && grad && !gather) v2A = v2B = pair_launch = false;   // (the loss passes form the gradients on their way)
  PassPlans qa, qb;
  if ((rc = plan_passes(K, ga, A->rows, A->cols, grad, &qa, v2A, asym, pair_launch ? 2 : 1, gather))) return rc;
  if ((rc = plan_passes(K, gb, B->cols, B->rows, grad, &qb, v2B, asym, pair_launch ? 2 : 1, gather))) return rc;
  const CorePlan &pa = qa.first, &pb = qb.first;
  {
    const size_t la = core_lds_bytes(K, ga.Gk, qa.fused), lb = core_lds_bytes(K, gb.Gk, qb.fused);
    if (la == 0 || lb == 0 || la > kLdsLimit || lb > kLdsLimit) return CAFEQ_ERR_UNSUPPORTED;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  DualWs w = carve_dual(ws, qa, qb, nb, grad);
  const QGrid grid = grid_for(cfg);
  // float16 forward operands: passes over prepared weights, and the gradient-free general pass over blocks of 128 (one block per segment)
  const bool f16A = v2A || core_forward_f16(K, ga.Gk, cfg->bits), f16B = v2B || core_forward_f16(K, gb.Gk, cfg->bits);

  // (passes that split their operands themselves: no planes, and every header is written by them)
  if (!(pair_launch && v2_splits_planes(K, true, false)) && !(qa.core32 && qb.core32)) {
    const SplitRequest req[4] = {{x->T, w.a.pfwd, 1, v2A ? v2_fwd_parts(K) : f16A ? 2 : kFwdPlanes, f16A ? w.a.fs : nullptr, v2A ? 1 : 0, v2A ? 4 : 14},
                                 {x->Tinv, w.a.pinv, 1, kInvPlanes, v2A ? w.a.fsi : nullptr, 0, 4},
                                 {x->Tinv, w.b.pfwd, 0, v2B ? v2_fwd_parts(K) : f16B ? 2 : kFwdPlanes, f16B ? w.b.fs : nullptr, v2B ? 1 : 0, v2B ? 4 : 14},
                                 {x->T, w.b.pinv, 0, kInvPlanes, v2B ? w.b.fsi : nullptr, 0, 4}};
    // (of the members whose pass reads planes)
    const int first = qa.core32 ? 2 : 0, last = qb.core32 ? 2 : 4;
    if ((rc = launch_split_planes_multi(req + first, last - first, K, nb, st, w.hdrA, pa.nslot + pb.nslot))) return rc;
  }
  // Each member: the loss pass, then (two-pass gradient) straight away the gradient pass over
  // the same weights, while they are still in the memory-side cache.  The gradient pass takes
  // its exponentials relative to the member's own largest group maximum; the final reduction
  // rescales to the pair's.
  CoreParams a, ag, b, bg;
  fill_common(&a, A, pa, 1);
  a.Afwd = w.a.pfwd; a.Ainv = w.a.pinv;
  a.grid = grid; a.do_inverse = 1; a.do_grad = qa.fused ? 1 : 0; a.loss_kind = kLossLse; a.lse_t = lse_t;
  a.codes = codesU; a.scales = scalesU; a.slot_grad = w.a.slot_grad; a.slot_hdr = w.hdrA;
  a.fscale = f16A ? w.a.fs : nullptr; a.fscale_inv = v2A ? w.a.fsi : nullptr;
  a.asym = asym ? 1 : 0;
  a.mins = asym && scalesU ? scalesU + A->rows * (A->cols / ga.G) : nullptr;   // the minima follow the scales
  fill_common(&b, B, pb, x->rep);
  b.Afwd = w.b.pfwd; b.Ainv = w.b.pinv;
  b.grid = grid; b.do_inverse = 1; b.do_grad = qb.fused ? 1 : 0; b.loss_kind = kLossLse; b.lse_t = lse_t;
  b.codes = codesV; b.scales = scalesV; b.slot_grad = w.b.slot_grad; b.slot_hdr = w.hdrB;
  b.fscale = f16B ? w.b.fs : nullptr; b.fscale_inv = v2B ? w.b.fsi : nullptr;
  b.asym = asym ? 1 : 0;
  b.mins = asym && scalesV ? scalesV + (B->rows / gb.G) * B->cols : nullptr;
  a.Tfwd = b.Tback = x->T;
  a.Tback = b.Tfwd = x->Tinv;
  const cafeq_mat* mats[2] = {A, B};
  const PassPlans* pps[2] = {&qa, &qb};
  const bool owner = grad && !gather && grad_owner_eligible(mats, pps, 2, K, x->rep);

  if (pair_launch) {
    set_prepared(&a, A, CAFEQ_AXIS_COL);
    set_prepared(&b, B, CAFEQ_AXIS_ROW);
    a.rec = qa.two ? w.a.rec : nullptr;
    b.rec = qb.two ? w.b.rec : nullptr;
    if ((rc = launch_loss_prepared_pair(K, ga.Gk, a, b, st))) return rc;
  } else if ((rc = run_core(K, CAFEQ_AXIS_COL, ga, a, w.a.rec, w.a.grec, qa.two, st, v2A ? A : nullptr, w.a.rec_mm,
                            w.a.grec_mm, w.a.zkeep, qa.core32))) {
    return rc;
  }
  ag = a;
  if (!gather && !owner && qa.two && (rc = run_grad_pass(K, CAFEQ_AXIS_COL, A, 1, qa, w.a, kLossLse, 0.f, lse_t, w.hdrA, int(pa.nslot),
                                              w.member_ref, &ag, st)))
    return rc;
  if (!pair_launch && (rc = run_core(K, CAFEQ_AXIS_ROW, gb, b, w.b.rec, w.b.grec, qb.two, st, v2B ? B : nullptr, w.b.rec_mm,
                                     w.b.grec_mm, w.b.zkeep, qb.core32)))
    return rc;
  bg = b;
  if (!gather && !owner && qb.two && (rc = run_grad_pass(K, CAFEQ_AXIS_ROW, B, x->rep, qb, w.b, kLossLse, 0.f, lse_t, w.hdrB, int(pb.nslot),
                                              w.member_ref + 1, &bg, st)))
    return rc;

  const int64_t ngroups = A->rows * (A->cols / ga.G) + (B->rows / gb.G) * B->cols;
  if (!owner && !(grad && gather) && (rc = launch_reduce_losses(kLossLse, w.hdrA, int(pa.nslot), w.hdrB, int(pb.nslot), 0.f, lse_t, ngroups,
                                           losses, w.lse_ms, st)))
    return rc;
  if (grad && gather) {
    // both members' gradients row by row from the records; d/dT = -P^T G_P P^T follows
    const GradGatherJob jobs[2] = {grad_gather_job(A, CAFEQ_AXIS_COL, nb, 1, qa, w.a, gradT, 1),
                                   grad_gather_job(B, CAFEQ_AXIS_ROW, nb, x->rep, qb, w.b, w.gp, 0)};
    LossArgs la{};
    la.hdrA = w.hdrA; la.nslotA = int(pa.nslot); la.hdrB = w.hdrB; la.nslotB = int(pb.nslot); la.kind = kLossLse;
    la.t = lse_t; la.ngroups = ngroups; la.losses = losses; la.lse_ms = w.lse_ms;
    if ((rc = launch_grad_gather_timed(K, jobs, 2, la, nullptr, st))) return rc;
    if ((rc = launch_bgemm_chain(x->Tinv, w.gp, w.x1, gradT, K, nb, -1.f, 1.f, st, hook))) return rc;
  } else if (grad && owner) {
    // both members' gradient passes in one launch: one workgroup per block writes member A's share into gradT
    // (transposed) and member B's G_P; d/dT = -P^T G_P P^T follows.  The pair's LogSumExp has to be known to
    // them: every workgroup reduces the partial headers itself, the first also writes the losses.
    const GradOwnerJob jobs[2] = {grad_owner_job(A, CAFEQ_AXIS_COL, qa, w.a, gradT, 1),
                                  grad_owner_job(B, CAFEQ_AXIS_ROW, qb, w.b, w.gp, 0)};
    LossArgs la{};
    la.hdrA = w.hdrA; la.nslotA = int(pa.nslot); la.hdrB = w.hdrB; la.nslotB = int(pb.nslot); la.kind = kLossLse;
    la.t = lse_t; la.ngroups = ngroups; la.losses = losses; la.lse_ms = w.lse_ms;
    if ((rc = launch_grad_owner_timed(jobs, 2, kLossLse, 0.f, lse_t, w.lse_ms, st, &la))) return rc;
    if ((rc = launch_bgemm_chain(x->Tinv, w.gp, w.x1, gradT, K, nb, -1.f, 1.f, st, hook))) return rc;
  } else if (grad) {
    // member A into gradT; member B: G_P of transform block b sums its rep row-blocks; d/dT = -P^T G_P P^T
    if ((rc = launch_reduce_grad_pair(ag, ga.Gk, qa.fused, qa.two ? w.member_ref : nullptr, gradT, bg, gb.Gk, qb.fused,
                                      qb.two ? w.member_ref + 1 : nullptr, w.gp, K, nb, w.lse_ms, st)))
      return rc;
    if ((rc = launch_bgemm_chain(x->Tinv, w.gp, w.x1, gradT, K, nb, -1.f, 1.f, st, hook))) return rc;
  }
  return CAFEQ_OK;
}

int cafeq_dual_proxy_loss_fwd_bwd(const cafeq_mat* A, const cafeq_mat* B, const cafeq_xform* x,
                                  const cafeq_quant_cfg* cfg, float lse_t, float* losses, float* gradT,
                                  int8_t* codesU, float* scalesU, int8_t* codesV, float* scalesV,
                                  void* ws, void* stream) {
  return dual_impl(A, B, x, cfg, lse_t, losses, gradT, codesU, scalesU, codesV, scalesV, ws, stream, nullptr);
}

// The correction's operand planes; for xform256.hip (blocks of 256, groups inside the block) of what it adds to the identity
static int split_correction(const AdaptiveWs& w, int k, int nb, const GroupPlan& gp, CoreParams* p, hipStream_t st) {
  const SplitRequest req{w.Cmat, w.planes, 0, kFwdPlanes, nullptr, 0, 14, k == 256 && gp.gspan == 1};
  p->Afwd = w.planes; p->Ainv = nullptr;
  return launch_split_planes_multi(&req, 1, k, nb, st);
}

int cafeq_adaptive_round_step(const float* U, const float* V, int64_t rowsA, int64_t colsA, int64_t rowsB,
                              int64_t colsB, const cafeq_quant_cfg* cfg, int k, int nb, int rep, int half,
                              int8_t* codesU, float* scalesU, int8_t* codesV, float* scalesV, int* status,
                              void* ws, void* stream) {
  int rc = check_cfg(cfg, false);
  if (rc) return rc;
  if (!U || !V || !codesU || !scalesU || !codesV || !scalesV) return CAFEQ_ERR_INVALID_ARG;
  if (half < 0 || half > 2) return CAFEQ_ERR_INVALID_ARG;
  if (!supported_block(k)) return CAFEQ_ERR_UNSUPPORTED;
  if (nb <= 0 || rep <= 0 || rowsA <= 0 || colsB <= 0) return CAFEQ_ERR_BAD_SHAPE;
  if (colsA != int64_t(nb) * k || rowsB != int64_t(nb) * rep * k || colsB % 4 != 0) return CAFEQ_ERR_BAD_SHAPE;
  if (!aligned16(U) || !aligned16(V) || !aligned16(codesU) || !aligned16(codesV) || !aligned16(scalesU) ||
      !aligned16(scalesV))
    return CAFEQ_ERR_BAD_ALIGN;
  if (!ws) return CAFEQ_ERR_WORKSPACE;
  AdaptivePlan ap;
  if ((rc = plan_adaptive(cfg, k, nb, rep, rowsA, colsA, rowsB, colsB, &ap))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const AdaptiveWs w = carve_adaptive(ws, ap, k, nb, nullptr);
  const QGrid grid = make_grid(cfg->bits);

  if (half == 0 || half == 1) {
    // line 3: C = pinv(Uq_b) U_b per head, Vq <- Q(C V_q)
    if ((rc = launch_gram_pair(CAFEQ_AXIS_COL, U, codesU, scalesU, rowsA, colsA, k, ap.ga.G, nb, 1, ap.chunkA,
                               ap.nchunkA, w.partial, st)))
      return rc;
    if ((rc = launch_gj_solve(k, nb, ap.nchunkA, w.partial, w.work, w.Sinv, w.Rsum, w.Cmat, status, 2, 0, st))) return rc;
    cafeq_mat mv{V, rowsB, colsB, colsB, CAFEQ_F32};
    CoreParams p;
    fill_common(&p, &mv, ap.planV, rep);
    if ((rc = split_correction(w, k, nb, ap.gb, &p, st))) return rc;
    p.grid = grid; p.codes = codesV; p.scales = scalesV;
    if ((rc = run_core(k, CAFEQ_AXIS_ROW, ap.gb, p, w.rec, w.grec, false, st))) return rc;
  }
  if (half == 0 || half == 2) {
    // line 4: C^T = V_[b] pinv(Vq_[b]) per head, Uq_b <- Q(U_b C^T)
    if ((rc = launch_gram_pair(CAFEQ_AXIS_ROW, V, codesV, scalesV, rowsB, colsB, k, ap.gb.G, nb, rep, ap.chunkB,
                               ap.nchunkB, w.partial, st)))
      return rc;
    if ((rc = launch_gj_solve(k, nb, rep * ap.nchunkB, w.partial, w.work, w.Sinv, w.Rsum, w.Cmat, status, 2, 1, st))) return rc;
    cafeq_mat mu{U, rowsA, colsA, colsA, CAFEQ_F32};
    CoreParams p;
    fill_common(&p, &mu, ap.planU, 1);
    if ((rc = split_correction(w, k, nb, ap.ga, &p, st))) return rc;
    p.grid = grid; p.codes = codesU; p.scales = scalesU;
    if ((rc = run_core(k, CAFEQ_AXIS_COL, ap.ga, p, w.rec, w.grec, false, st))) return rc;
  }
  return CAFEQ_OK;
}

}  // extern "C"
