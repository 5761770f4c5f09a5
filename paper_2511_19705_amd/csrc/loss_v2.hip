// The weights' prepared copies, and the loss pass over them (loss_v2.hpp) for blocks of 128.
#include "loss_v2.hpp"

namespace cafeq {

namespace {

// ---------------------------------------------------------------------------------------------------
// preparation: one workgroup per tile of 32 lines x 128 axis indices
// ---------------------------------------------------------------------------------------------------
struct PrepArgs {
  const void* W; int dtype; int64_t rows, cols, ld; int axis;
  int64_t nlines, nlp; int nseg;
  unsigned char* planes; float* lscale; double* partial;
  unsigned char* lines;   // line-major copy (may be null)
};

__global__ __launch_bounds__(256) void prepare_tiles_kernel(const PrepArgs a) {
  __shared__ float tile[32][129];
  __shared__ double red[4];
  const int64_t nstrip = a.nlp / 32;
  const int64_t tix = blockIdx.x;
  const int seg = int(tix / nstrip);
  const int64_t strip = tix - int64_t(seg) * nstrip;
  const int t = threadIdx.x;
  for (int r = 0; r < 16; ++r) {
    const int idx = r * 256 + t;
    int li, m;
    if (a.axis == CAFEQ_AXIS_COL) { li = idx >> 7; m = idx & 127; } else { m = idx >> 5; li = idx & 31; }
    const int64_t line = strip * 32 + li, ax = int64_t(seg) * 128 + m;
    float v = 0.f;
    if (line < a.nlines) {
      const int64_t off = a.axis == CAFEQ_AXIS_COL ? line * a.ld + ax : ax * a.ld + line;
      v = a.dtype == CAFEQ_F32 ? static_cast<const float*>(a.W)[off]
                               : bf16_bits_to_f32(static_cast<const uint16_t*>(a.W)[off]);
    }
    tile[li][m] = v;
  }
  __syncthreads();
  if (a.lines) {
    // (a bfloat16's bits are the upper half of its float32's)
    for (int r = 0; r < 4; ++r) {
      const int li = r * 8 + (t >> 5), m = 4 * (t & 31);
      const int64_t at = (int64_t(seg) * a.nlp + strip * 32 + li) * 128 + m;
      const float* s = &tile[li][m];
      if (a.dtype == CAFEQ_F32) {
        *reinterpret_cast<float4*>(a.lines + at * 4) = make_float4(s[0], s[1], s[2], s[3]);
      } else {
        *reinterpret_cast<uint2*>(a.lines + at * 2) =
            make_uint2(__float_as_uint(s[0]) >> 16 | (__float_as_uint(s[1]) & 0xFFFF0000u),
                       __float_as_uint(s[2]) >> 16 | (__float_as_uint(s[3]) & 0xFFFF0000u));
      }
    }
  }
  const int li = t >> 3, c = t & 7;
  float x[16];
  float mx = 0.f;
  double sq = 0;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    x[e] = tile[li][16 * c + e];
    // (an infinity must not set the scale: the line's other blocks of 32 or 64 would be scaled away)
    if (fabsf(x[e]) < INFINITY) mx = fmaxf(mx, fabsf(x[e]));
    sq += double(x[e]) * x[e];
  }
  const int parts = prepared_parts(a.dtype);
  mx = fmaxf(mx, __shfl_xor(mx, 1));
  const float mx32 = mx;
  mx = fmaxf(mx, __shfl_xor(mx, 2));
  const float mx64 = mx;
  mx = fmaxf(mx, __shfl_xor(mx, 4));
  int ex = int(__float_as_uint(mx) >> 23);
  ex = ex < 4 ? 4 : (ex > 254 ? 254 : ex);          // (the scale and the factor back stay normal numbers)
  const float wsc = __uint_as_float(uint32_t(257 - ex) << 23);          // 2^(3 - (ex - 127)): largest magnitude in [2^3, 2^4)
  // 32 or 64 inputs that are so much smaller than the segment's largest that their parts end before their bits do (the second
  // part at 2^-24; bfloat16's eight bits end long before): marked in the line's scale (rescale_strip, loss_v2.hpp)
  const float least = mx * (parts == 2 ? 0x1p-5f : 0x1p-8f);
  uint32_t far = (mx32 > 0.f && mx32 < least ? kFar32 : 0u) | (mx64 > 0.f && mx64 < least ? kFar64 : 0u);
  far |= __shfl_xor(far, 2);
  far |= __shfl_xor(far, 4);
  if (c == 0) a.lscale[int64_t(seg) * a.nlp + strip * 32 + li] = __uint_as_float(uint32_t(ex - 3) << 23 | far);
  unsigned char* tp = a.planes + tix * int64_t(v2_tile_bytes(parts)) + c * 1024 * parts;
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      uint32_t hb[2], lb[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        weight_parts(x[8 * hh + 2 * e2 + u] * wsc, parts == 1, &hb[u], &lb[u]);
      }
      hi[e2] = hb[0] | (hb[1] << 16);
      lo[e2] = lb[0] | (lb[1] << 16);
    }
    *reinterpret_cast<uint4*>(tp + (hh * 32 + li) * 16) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    if (parts == 2) *reinterpret_cast<uint4*>(tp + 1024 + (hh * 32 + li) * 16) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
  }
  sq = wave_sum(sq);
  if ((t & 63) == 0) red[t >> 6] = sq;
  __syncthreads();
  if (t == 0) a.partial[tix] = red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(256) void prepare_sum_kernel(const double* __restrict__ partial, int64_t n,
                                                           float* __restrict__ out) {
  __shared__ double red[256];
  double t = 0;
  for (int64_t i = threadIdx.x; i < n; i += 256) t += partial[i];
  red[threadIdx.x] = t;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = float(red[0]);
}

}  // namespace

PreparedLayout prepared_layout(int64_t nlines, int64_t naxis, int dtype, int axis) {
  PreparedLayout l;
  l.nlp = (nlines + kV2MacroLines - 1) / kV2MacroLines * kV2MacroLines;
  l.nseg = naxis / 128;
  l.ntiles = l.nseg * (l.nlp / 32);
  l.off_lscale = 256;
  l.off_planes = align_up(l.off_lscale + size_t(l.nseg) * l.nlp * sizeof(float), 256);
  l.off_partial = l.off_planes + size_t(l.ntiles) * v2_tile_bytes(prepared_parts(dtype));
  l.off_gtiles = align_up(l.off_partial + size_t(l.ntiles) * sizeof(double), 256);
  l.off_lines = align_up(l.off_gtiles + prepared_gtiles_bytes(nlines, naxis, dtype), 256);
  const size_t lines = axis == CAFEQ_AXIS_ROW ? size_t(l.nseg) * l.nlp * 128 * (dtype == CAFEQ_BF16 ? 2 : 4) : 0;
  l.bytes = align_up(l.off_lines + lines, 256);
  return l;
}

int launch_prepare(const cafeq_mat* W, int axis, void* prepared, hipStream_t st) {
  const bool col = axis == CAFEQ_AXIS_COL;
  const int64_t nlines = col ? W->rows : W->cols, naxis = col ? W->cols : W->rows;
  if (naxis % 128 != 0) return CAFEQ_ERR_BAD_SHAPE;
  const PreparedLayout l = prepared_layout(nlines, naxis, W->dtype, axis);
  unsigned char* base = static_cast<unsigned char*>(prepared);
  PrepArgs a;
  a.W = W->data; a.dtype = W->dtype; a.rows = W->rows; a.cols = W->cols; a.ld = W->ld; a.axis = axis;
  a.nlines = nlines; a.nlp = l.nlp; a.nseg = int(l.nseg);
  a.planes = base + l.off_planes; a.lscale = reinterpret_cast<float*>(base + l.off_lscale);
  a.partial = reinterpret_cast<double*>(base + l.off_partial);
  a.lines = col ? nullptr : base + l.off_lines;
  hipLaunchKernelGGL(prepare_tiles_kernel, dim3(unsigned(l.ntiles)), dim3(256), 0, st, a);
  CAFEQ_CHECK_LAUNCH();
  hipLaunchKernelGGL(prepare_sum_kernel, dim3(1), dim3(256), 0, st, a.partial, l.ntiles, reinterpret_cast<float*>(base));
  CAFEQ_CHECK_LAUNCH();
  return launch_prepare_gtiles(W, axis, base + l.off_gtiles, st);
}

// Both members of a pair (member A on its columns, member B on its rows) in one launch; same group length and
// the same choice of records for both, no codes or scales.
int launch_loss_v2_pair(int K, int G, const CoreParams& pa, const CoreParams& pb, hipStream_t st) {
  for (const CoreParams* p : {&pa, &pb})
    if (!p->prep_planes || !p->prep_lscale || !p->prep_wsq || !p->slot_hdr || p->codes || p->scales || p->loss_kind != kLossLse ||
        (v2_splits_planes(K, true, false) ? !p->Tfwd || !p->Tback : !p->fscale || !p->fscale_inv))
      return CAFEQ_ERR_INVALID_ARG;
  if ((pa.rec != nullptr) != (pb.rec != nullptr)) return CAFEQ_ERR_INVALID_ARG;
  switch (K) {
    case 32: return launch_loss_v2_pair_k32(G, pa, pb, st);
    case 64: return launch_loss_v2_pair_k64(G, pa, pb, st);
    case 128: return launch_v2_pair_k<128>(G, pa, pb, st);
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
}

int launch_loss_v2(int K, int G, int axis, const CoreParams& p, hipStream_t st) {
  if (!p.prep_planes || !p.prep_lscale || !p.prep_wsq || !p.slot_hdr ||
      (v2_splits_planes(K, false, p.codes || p.scales) ? !p.Tfwd || !p.Tback || (p.loss_kind == kLossSur && !p.rG_out) : !p.fscale || !p.fscale_inv))
    return CAFEQ_ERR_INVALID_ARG;
  switch (K) {
    case 32: return launch_loss_v2_k32(G, axis, p, st);
    case 64: return launch_loss_v2_k64(G, axis, p, st);
    case 128: return launch_v2_k<128>(G, axis, p, st);
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
}

}  // namespace cafeq
