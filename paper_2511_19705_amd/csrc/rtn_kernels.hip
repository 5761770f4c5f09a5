// Per-group absmax round-to-nearest without a transform (the HBM-bound stage).
//
// Rounding rule of the paper's Eq. (1) (nearest integer) on the symmetric grid
// described in cafeq.h.  Algorithmic traffic per element: one read (4 B float32 /
// 2 B bfloat16), one int8 code written, 4/g bytes of scale.
//
// The kernels:
//   rtn_col_fast : groups along the contiguous axis, g = 4 * 2^n <= 256.  One lane owns
//                  four (float32) or sixteen (bfloat16) consecutive elements, adjacent lanes
//                  own a group; the absmax is an all-reduce over that lane cluster with DPP
//                  (inside a 16-lane row) and LDS-crossbar shuffles (across rows).
//   rtn_row_fast : groups along the strided axis, g = 16 * {1,2,4,8,16}.  A workgroup of
//                  g/16 waves owns g rows x 256 columns; each wave keeps 16 rows of four
//                  columns per lane in registers, column maxima are combined through LDS,
//                  so the tile is read from memory once.
//   rtn_col_long : groups of 2048 and more (whole channels) kept in a workgroup's registers.
//   rtn_col_vec, rtn_col_any / rtn_row_any : any group length dividing the line, two passes per group.
// The squared-error output is reduced in two fixed-order stages (per-workgroup partials
// in the caller's workspace, then one workgroup), so it is reproducible run to run.
#include "cafeq_common.hpp"
#include "cafeq_internal.hpp"

namespace cafeq {

namespace {

constexpr int kColThreads = 256;
constexpr int kColUnroll = 4;

__device__ __forceinline__ void block_store_partial(float err, double* partial) {
  __shared__ double red[16];
  double e = wave_sum(double(err));
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (lane == 0) red[wave] = e;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0;
    const int nw = (blockDim.x + kWave - 1) / kWave;
    for (int i = 0; i < nw; ++i) t += red[i];
    partial[blockIdx.y * size_t(gridDim.x) + blockIdx.x] = t;
  }
}

// The grid of a call: symmetric (p0 = qmax, p1 = qmin) or the min/max grid of the paper's Eq. (1) (p0 = levels).
// Min/max, in single precision: r = fl(max - min), inv = min(fl(levels / r), FLT_MAX) (0 for a constant group),
// q = clamp(rint(fl(fl(z - min) * inv)), 0, levels), s = fl(r / levels), dequantized fl(fl(q * s) + min);
// levels = 2^b - 1.
__device__ __forceinline__ float mm_inv(float r, float levels) {
  return r > 0.f ? fminf(__fdiv_rn(levels, r), FLT_MAX) : 0.f;
}
// v = scaled value, clamped to the grid (a NaN to its lower end) and rounded to nearest even: adding 1.5 2^23 leaves
// the integer in the low mantissa bits, so the sum's low byte is the code and the sum less 1.5 2^23 the code as a float
constexpr float kRoundMagic = 12582912.f;
__device__ __forceinline__ float code_bits(float v, float lo, float hi) {
  return __fadd_rn(__builtin_amdgcn_fmed3f(v, lo, hi), kRoundMagic);
}
__device__ __forceinline__ uint32_t pack_code_bits(float m0, float m1, float m2, float m3) {
  const uint32_t lo = __builtin_amdgcn_perm(__float_as_uint(m1), __float_as_uint(m0), 0x0C0C0400u);
  const uint32_t hi = __builtin_amdgcn_perm(__float_as_uint(m3), __float_as_uint(m2), 0x04000C0Cu);
  return lo | hi;
}

// EPL consecutive elements as loaded
typedef uint32_t raw4 __attribute__((ext_vector_type(4)));
template <typename Tag, int EPL>
struct RawElems;
template <int EPL>
struct RawElems<F32Tag, EPL> {
  raw4 w[EPL / 4];
  __device__ __forceinline__ void load(const float* p) {
#pragma unroll
    for (int q = 0; q < EPL / 4; ++q) w[q] = reinterpret_cast<const raw4*>(p)[q];
  }
  __device__ __forceinline__ float get(int e) const { return __uint_as_float(w[e / 4][e % 4]); }
};
template <int EPL>
struct RawElems<BF16Tag, EPL> {
  uint32_t w[EPL / 2];
  __device__ __forceinline__ void load(const uint16_t* p) {
    if constexpr (EPL >= 8) {
#pragma unroll
      for (int q = 0; q < EPL / 8; ++q) {
        const raw4 v = reinterpret_cast<const raw4*>(p)[q];
        w[4 * q] = v[0]; w[4 * q + 1] = v[1]; w[4 * q + 2] = v[2]; w[4 * q + 3] = v[3];
      }
    } else {
      const uint2 v = *reinterpret_cast<const uint2*>(p);
      w[0] = v.x; w[1] = v.y;
    }
  }
  __device__ __forceinline__ float get(int e) const {
    return __uint_as_float(e % 2 ? w[e / 2] & 0xFFFF0000u : w[e / 2] << 16);
  }
};

// Groups along the contiguous axis: a lane owns EPL consecutive elements, LPG adjacent lanes a group (g = EPL * LPG, a
// power of two), U such pieces of a lane are in flight at once.  (Fewer workgroups striding over the matrix leave fewer
// partials of the squared error but run 8 % slower: 46.5 against 42 us in float32.)
// float32: four elements per lane (one 128-bit load), bound by HBM: 42 us on three 3584 x 14336 matrices in turn, 6.1 TB/s.
// bfloat16: half the bytes per element, so with four elements per lane the two divisions, the group reduction (through
// LDS for 32 lanes) and the packing bound it (39.9 us on 3584 x 14336 with groups of 128, 3.9 TB/s); sixteen elements per
// lane share them, the reduction stays inside a row of 16 lanes, and a code costs five instructions instead of nine:
// 27.4 us, 5.6 TB/s.
template <typename Tag, int EPL, int LPG, int U, bool DENSE, bool MM>
__global__ __launch_bounds__(kColThreads) void rtn_col_fast(
    const typename Tag::elem* __restrict__ W, uint32_t nvec, uint32_t colsv, int64_t ld, float p0, float p1,
    uint32_t* __restrict__ codes, float* __restrict__ scales, float* __restrict__ mins, double* __restrict__ partial) {
  float err = 0.f;
  const uint32_t base = blockIdx.x * (kColThreads * U) + threadIdx.x;
  RawElems<Tag, EPL> raw[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const uint32_t v = base + j * kColThreads;
    size_t off;
    const uint32_t vv = v < nvec ? v : nvec - 1;     // (a group lies wholly inside or outside the matrix)
    if constexpr (DENSE) {
      off = size_t(vv) * EPL;
    } else {
      const uint32_t r = vv / colsv;
      off = size_t(r) * ld + size_t(vv - r * colsv) * EPL;
    }
    raw[j].load(W + off);
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const uint32_t v = base + j * kColThreads;
    const bool live = v < nvec;
    float inv, s, lo = 0.f;
    if constexpr (MM) {
      float hi = raw[j].get(0), nlo = -hi;           // -min, so that one kind of reduction serves both
#pragma unroll
      for (int e = 1; e < EPL; ++e) {
        hi = fmaxf(hi, raw[j].get(e));
        nlo = fmaxf(nlo, -raw[j].get(e));
      }
      hi = cluster_allmax<LPG>(hi);
      nlo = cluster_allmax<LPG>(nlo);
      lo = -nlo;
      const float r = __fsub_rn(hi, lo);
      inv = mm_inv(r, p0);
      s = __fdiv_rn(r, p0);
    } else {
      float a = fabsf(raw[j].get(0));
#pragma unroll
      for (int e = 1; e < EPL; ++e) a = fmaxf(a, fabsf(raw[j].get(e)));
      a = cluster_allmax<LPG>(a);
      inv = grid_inv(a, p0);
      s = grid_scale(a, p0);
    }
    uint32_t c[EPL / 4];
    float e2 = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; e += 4) {
      float m[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float z = raw[j].get(e + i);
        m[i] = MM ? code_bits(__fmul_rn(__fsub_rn(z, lo), inv), 0.f, p0) : code_bits(__fmul_rn(z, inv), p1, p0);
        if (partial) {                               // uniform over the launch
          const float zq = __fmul_rn(__fsub_rn(m[i], kRoundMagic), s);
          const float d = (MM ? __fadd_rn(zq, lo) : zq) - z;
          e2 = fmaf(d, d, e2);
        }
      }
      c[e / 4] = pack_code_bits(m[0], m[1], m[2], m[3]);
    }
    if (live) {
      if constexpr (EPL == 16) {
        const raw4 o = {c[0], c[1], c[2], c[3]};
        reinterpret_cast<raw4*>(codes)[v] = o;
      } else {
        codes[v] = c[0];
      }
      if ((threadIdx.x % LPG) == 0) {
        if (scales) scales[v / LPG] = s;
        if (MM && mins) mins[v / LPG] = lo;
      }
      err += e2;
    }
  }
  if (partial) block_store_partial(err, partial);
}

// Long groups along the contiguous axis (2048 elements and more: whole channels), one workgroup per group, which keeps the
// group in registers between the reduction and the rounding: every lane NP pieces of 16 bytes, a workgroup's width apart.
// One read of the matrix instead of two (rtn_col_vec, one wave per group and one request at a time): whole channels of
// 3584 x 14336 in bfloat16 63 -> 26 us, in float32 85 -> 44 us.
template <typename Tag, int NP, bool MM>
__global__ __launch_bounds__(1024) void rtn_col_long(
    const typename Tag::elem* __restrict__ W, int64_t gpr, int64_t ngroups, int64_t cols, int64_t ld, int g, float p0, float p1,
    int8_t* __restrict__ codes, float* __restrict__ scales, float* __restrict__ mins, double* __restrict__ partial) {
  constexpr int PE = Tag::dtype == CAFEQ_BF16 ? 8 : 4;
  __shared__ float red[2][2][16];
  const int nt = blockDim.x, nw = nt / kWave, wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  float err = 0.f;
  int turn = 0;
  for (int64_t gi = blockIdx.x; gi < ngroups; gi += gridDim.x, turn ^= 1) {
    const int64_t r = gi / gpr, c0 = (gi - r * gpr) * g;
    const typename Tag::elem* src = W + r * ld + c0;
    int8_t* dst = codes + r * cols + c0;
    RawElems<Tag, PE> raw[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int i = (int(threadIdx.x) + q * nt) * PE;
      raw[q].load(src + (i < g ? i : g - PE));        // (past the end: the last piece again, which changes no maximum)
    }
    float hi = MM ? -FLT_MAX : 0.f, nlo = -FLT_MAX;
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int e = 0; e < PE; ++e) {
        const float z = raw[q].get(e);
        hi = fmaxf(hi, MM ? z : fabsf(z));
        if (MM) nlo = fmaxf(nlo, -z);
      }
    hi = cluster_allmax<64>(hi);
    if (MM) nlo = cluster_allmax<64>(nlo);
    if (lane == 0) { red[turn][0][wave] = hi; red[turn][1][wave] = nlo; }
    __syncthreads();                                  // (two sets of slots: the next group's do not meet this one's readers)
    hi = red[turn][0][0]; nlo = red[turn][1][0];
    for (int w = 1; w < nw; ++w) { hi = fmaxf(hi, red[turn][0][w]); nlo = fmaxf(nlo, red[turn][1][w]); }
    const float lo = MM ? -nlo : 0.f, range = MM ? __fsub_rn(hi, lo) : hi;
    const float inv = MM ? mm_inv(range, p0) : grid_inv(hi, p0), s = __fdiv_rn(range, p0);
    if (threadIdx.x == 0) {
      if (scales) scales[gi] = s;
      if (MM && mins) mins[gi] = lo;
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int i = (int(threadIdx.x) + q * nt) * PE;
      if (i < g) {
#pragma unroll
        for (int e = 0; e < PE; e += 4) {
          float m[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float z = raw[q].get(e + k);
            m[k] = MM ? code_bits(__fmul_rn(__fsub_rn(z, lo), inv), 0.f, p0) : code_bits(__fmul_rn(z, inv), p1, p0);
            if (partial) {
              const float zq = __fmul_rn(__fsub_rn(m[k], kRoundMagic), s);
              const float d = (MM ? __fadd_rn(zq, lo) : zq) - z;
              err = fmaf(d, d, err);
            }
          }
          *reinterpret_cast<uint32_t*>(dst + i + e) = pack_code_bits(m[0], m[1], m[2], m[3]);
        }
      }
    }
  }
  if (partial) block_store_partial(err, partial);
}

constexpr int kRowRPW = 16;  // rows per wave

template <typename Tag, int NW>
__global__ __launch_bounds__(NW * kWave) void rtn_row_fast(
    const typename Tag::elem* __restrict__ W, int64_t cols, int64_t ld, QGrid grid,
    int8_t* __restrict__ codes, float* __restrict__ scales, double* __restrict__ partial) {
  __shared__ float4 smax[NW][kWave];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int64_t c = int64_t(blockIdx.x) * 256 + lane * 4;
  const int64_t r0 = int64_t(blockIdx.y) * (NW * kRowRPW) + wave * kRowRPW;
  const bool live = c < cols;
  float4 x[kRowRPW];
  float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < kRowRPW; ++i) {
    x[i] = live ? load4(W + (r0 + i) * ld + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    m.x = fmaxf(m.x, fabsf(x[i].x));
    m.y = fmaxf(m.y, fabsf(x[i].y));
    m.z = fmaxf(m.z, fabsf(x[i].z));
    m.w = fmaxf(m.w, fabsf(x[i].w));
  }
  if constexpr (NW > 1) {
    smax[wave][lane] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 o = smax[w][lane];
      m.x = fmaxf(m.x, o.x);
      m.y = fmaxf(m.y, o.y);
      m.z = fmaxf(m.z, o.z);
      m.w = fmaxf(m.w, o.w);
    }
  }
  const float4 inv = make_float4(grid_inv(m.x, grid.qmax), grid_inv(m.y, grid.qmax),
                                 grid_inv(m.z, grid.qmax), grid_inv(m.w, grid.qmax));
  const float4 s = make_float4(grid_scale(m.x, grid.qmax), grid_scale(m.y, grid.qmax),
                               grid_scale(m.z, grid.qmax), grid_scale(m.w, grid.qmax));
  float err = 0.f;
  if (live) {
    if (wave == 0 && scales) *reinterpret_cast<float4*>(scales + int64_t(blockIdx.y) * cols + c) = s;
#pragma unroll
    for (int i = 0; i < kRowRPW; ++i) {
      const float q0 = grid_code(x[i].x, inv.x, grid), q1 = grid_code(x[i].y, inv.y, grid);
      const float q2 = grid_code(x[i].z, inv.z, grid), q3 = grid_code(x[i].w, inv.w, grid);
      *reinterpret_cast<uint32_t*>(codes + (r0 + i) * cols + c) = pack4(q0, q1, q2, q3);
      if (partial) {
        const float e0 = __fmul_rn(q0, s.x) - x[i].x, e1 = __fmul_rn(q1, s.y) - x[i].y;
        const float e2 = __fmul_rn(q2, s.z) - x[i].z, e3 = __fmul_rn(q3, s.w) - x[i].w;
        err += e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3;
      }
    }
  }
  if (partial) block_store_partial(err, partial);
}

// One wave per group, group length a multiple of 4: 128-bit loads, four codes per store.
template <typename Tag>
__global__ __launch_bounds__(256) void rtn_col_vec(
    const typename Tag::elem* __restrict__ W, int64_t rows, int64_t cols, int64_t ld, int64_t g,
    QGrid grid, int8_t* __restrict__ codes, float* __restrict__ scales, double* __restrict__ partial) {
  const int lane = threadIdx.x % kWave;
  const int64_t gpr = cols / g, ngroups = rows * gpr;
  const int64_t wave0 = int64_t(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int64_t wstride = int64_t(gridDim.x) * (blockDim.x / kWave);
  float err = 0.f;
  for (int64_t gi = wave0; gi < ngroups; gi += wstride) {
    const int64_t r = gi / gpr, c0 = (gi - r * gpr) * g;
    const typename Tag::elem* src = W + r * ld + c0;
    float a = 0.f;
    for (int64_t i = int64_t(lane) * 4; i < g; i += kWave * 4) {
      const float4 z = load4(src + i);
      a = fmaxf(a, fmaxf(fmaxf(fabsf(z.x), fabsf(z.y)), fmaxf(fabsf(z.z), fabsf(z.w))));
    }
    a = cluster_allmax<64>(a);
    const float inv = grid_inv(a, grid.qmax), s = grid_scale(a, grid.qmax);
    if (lane == 0 && scales) scales[gi] = s;
    for (int64_t i = int64_t(lane) * 4; i < g; i += kWave * 4) {
      const float4 z = load4(src + i);
      const float q0 = grid_code(z.x, inv, grid), q1 = grid_code(z.y, inv, grid);
      const float q2 = grid_code(z.z, inv, grid), q3 = grid_code(z.w, inv, grid);
      *reinterpret_cast<uint32_t*>(codes + r * cols + c0 + i) = pack4(q0, q1, q2, q3);
      if (partial) {
        const float e0 = __fmul_rn(q0, s) - z.x, e1 = __fmul_rn(q1, s) - z.y;
        const float e2 = __fmul_rn(q2, s) - z.z, e3 = __fmul_rn(q3, s) - z.w;
        err += e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3;
      }
    }
  }
  if (partial) block_store_partial(err, partial);
}

// One wave per group, any group length.
template <typename Tag>
__global__ __launch_bounds__(256) void rtn_col_any(
    const typename Tag::elem* __restrict__ W, int64_t rows, int64_t cols, int64_t ld, int64_t g,
    QGrid grid, int8_t* __restrict__ codes, float* __restrict__ scales, double* __restrict__ partial) {
  const int lane = threadIdx.x % kWave;
  const int64_t gpr = cols / g, ngroups = rows * gpr;
  const int64_t wave0 = int64_t(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int64_t wstride = int64_t(gridDim.x) * (blockDim.x / kWave);
  float err = 0.f;
  for (int64_t gi = wave0; gi < ngroups; gi += wstride) {
    const int64_t r = gi / gpr, c0 = (gi - r * gpr) * g;
    const typename Tag::elem* src = W + r * ld + c0;
    float a = 0.f;
    for (int64_t i = lane; i < g; i += kWave) a = fmaxf(a, fabsf(load1(src + i)));
    a = cluster_allmax<64>(a);
    const float inv = grid_inv(a, grid.qmax), s = grid_scale(a, grid.qmax);
    if (lane == 0 && scales) scales[gi] = s;
    for (int64_t i = lane; i < g; i += kWave) {
      const float z = load1(src + i);
      const float q = grid_code(z, inv, grid);
      codes[r * cols + c0 + i] = int8_t(int(q));
      const float e = __fmul_rn(q, s) - z;
      err += e * e;
    }
  }
  if (partial) block_store_partial(err, partial);
}

// One thread per (group, column), any group length.
template <typename Tag>
__global__ __launch_bounds__(256) void rtn_row_any(
    const typename Tag::elem* __restrict__ W, int64_t rows, int64_t cols, int64_t ld, int64_t g,
    QGrid grid, int8_t* __restrict__ codes, float* __restrict__ scales, double* __restrict__ partial) {
  const int64_t total = (rows / g) * cols;
  float err = 0.f;
  for (int64_t id = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; id < total;
       id += int64_t(gridDim.x) * blockDim.x) {
    const int64_t gr = id / cols, c = id - gr * cols;
    const typename Tag::elem* src = W + gr * g * ld + c;
    float a = 0.f;
    for (int64_t i = 0; i < g; ++i) a = fmaxf(a, fabsf(load1(src + i * ld)));
    const float inv = grid_inv(a, grid.qmax), s = grid_scale(a, grid.qmax);
    if (scales) scales[id] = s;
    for (int64_t i = 0; i < g; ++i) {
      const float z = load1(src + i * ld);
      const float q = grid_code(z, inv, grid);
      codes[(gr * g + i) * cols + c] = int8_t(int(q));
      const float e = __fmul_rn(q, s) - z;
      err += e * e;
    }
  }
  if (partial) block_store_partial(err, partial);
}

// ---- the min/max grid of the paper's Eq. (1) ------------------------------------------------
__device__ __forceinline__ float mm_code(float z, float lo, float inv, float levels) {
  const float q = __builtin_rintf(__fmul_rn(__fsub_rn(z, lo), inv));
  return fminf(fmaxf(q, 0.f), levels);
}

// One wave per group along the contiguous axis, group length a multiple of 4 (whole channels
// included): 128-bit loads, four codes per 32-bit store; the second pass re-reads the group
// from cache.
template <typename Tag>
__global__ __launch_bounds__(256) void rtn_col_minmax_vec(
    const typename Tag::elem* __restrict__ W, int64_t rows, int64_t cols, int64_t ld, int64_t g, float levels,
    uint8_t* __restrict__ codes, float* __restrict__ scales, float* __restrict__ mins,
    double* __restrict__ partial) {
  const int lane = threadIdx.x % kWave;
  const int64_t gpr = cols / g, ngroups = rows * gpr;
  const int64_t wave0 = int64_t(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int64_t wstride = int64_t(gridDim.x) * (blockDim.x / kWave);
  float err = 0.f;
  for (int64_t gi = wave0; gi < ngroups; gi += wstride) {
    const int64_t r = gi / gpr, c0 = (gi - r * gpr) * g;
    const typename Tag::elem* src = W + r * ld + c0;
    float hi = -FLT_MAX, nlo = -FLT_MAX;
    for (int64_t i = int64_t(lane) * 4; i < g; i += kWave * 4) {
      const float4 z = load4(src + i);
      hi = fmaxf(hi, fmaxf(fmaxf(z.x, z.y), fmaxf(z.z, z.w)));
      nlo = fmaxf(nlo, fmaxf(fmaxf(-z.x, -z.y), fmaxf(-z.z, -z.w)));
    }
    hi = cluster_allmax<64>(hi);
    nlo = cluster_allmax<64>(nlo);
    const float lo = -nlo, rg = __fsub_rn(hi, lo);
    const float inv = mm_inv(rg, levels), s = __fdiv_rn(rg, levels);
    if (lane == 0) {
      if (scales) scales[gi] = s;
      if (mins) mins[gi] = lo;
    }
    for (int64_t i = int64_t(lane) * 4; i < g; i += kWave * 4) {
      const float4 z = load4(src + i);
      const float q0 = mm_code(z.x, lo, inv, levels), q1 = mm_code(z.y, lo, inv, levels);
      const float q2 = mm_code(z.z, lo, inv, levels), q3 = mm_code(z.w, lo, inv, levels);
      *reinterpret_cast<uint32_t*>(codes + r * cols + c0 + i) =
          uint32_t(q0) | (uint32_t(q1) << 8) | (uint32_t(q2) << 16) | (uint32_t(q3) << 24);
      if (partial) {
        const float e0 = __fadd_rn(__fmul_rn(q0, s), lo) - z.x, e1 = __fadd_rn(__fmul_rn(q1, s), lo) - z.y;
        const float e2 = __fadd_rn(__fmul_rn(q2, s), lo) - z.z, e3 = __fadd_rn(__fmul_rn(q3, s), lo) - z.w;
        err += e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3;
      }
    }
  }
  if (partial) block_store_partial(err, partial);
}

// One wave per group along the contiguous axis, any group length.
template <typename Tag>
__global__ __launch_bounds__(256) void rtn_col_minmax_any(
    const typename Tag::elem* __restrict__ W, int64_t rows, int64_t cols, int64_t ld, int64_t g, float levels,
    uint8_t* __restrict__ codes, float* __restrict__ scales, float* __restrict__ mins,
    double* __restrict__ partial) {
  const int lane = threadIdx.x % kWave;
  const int64_t gpr = cols / g, ngroups = rows * gpr;
  const int64_t wave0 = int64_t(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int64_t wstride = int64_t(gridDim.x) * (blockDim.x / kWave);
  float err = 0.f;
  for (int64_t gi = wave0; gi < ngroups; gi += wstride) {
    const int64_t r = gi / gpr, c0 = (gi - r * gpr) * g;
    const typename Tag::elem* src = W + r * ld + c0;
    float hi = -FLT_MAX, nlo = -FLT_MAX;
    for (int64_t i = lane; i < g; i += kWave) {
      const float z = load1(src + i);
      hi = fmaxf(hi, z);
      nlo = fmaxf(nlo, -z);
    }
    hi = cluster_allmax<64>(hi);
    nlo = cluster_allmax<64>(nlo);
    const float lo = -nlo, rg = __fsub_rn(hi, lo);
    const float inv = mm_inv(rg, levels), s = __fdiv_rn(rg, levels);
    if (lane == 0) {
      if (scales) scales[gi] = s;
      if (mins) mins[gi] = lo;
    }
    for (int64_t i = lane; i < g; i += kWave) {
      const float z = load1(src + i);
      const float q = mm_code(z, lo, inv, levels);
      codes[r * cols + c0 + i] = uint8_t(int(q));
      const float e = __fadd_rn(__fmul_rn(q, s), lo) - z;
      err += e * e;
    }
  }
  if (partial) block_store_partial(err, partial);
}

// One thread per (group, column): groups along the strided axis, any group length.
template <typename Tag>
__global__ __launch_bounds__(256) void rtn_row_minmax_any(
    const typename Tag::elem* __restrict__ W, int64_t rows, int64_t cols, int64_t ld, int64_t g, float levels,
    uint8_t* __restrict__ codes, float* __restrict__ scales, float* __restrict__ mins,
    double* __restrict__ partial) {
  const int64_t total = (rows / g) * cols;
  float err = 0.f;
  for (int64_t id = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; id < total;
       id += int64_t(gridDim.x) * blockDim.x) {
    const int64_t gr = id / cols, c = id - gr * cols;
    const typename Tag::elem* src = W + gr * g * ld + c;
    float hi = -FLT_MAX, lo = FLT_MAX;
    for (int64_t i = 0; i < g; ++i) {
      const float z = load1(src + i * ld);
      hi = fmaxf(hi, z);
      lo = fminf(lo, z);
    }
    const float rg = __fsub_rn(hi, lo);
    const float inv = mm_inv(rg, levels), s = __fdiv_rn(rg, levels);
    if (scales) scales[id] = s;
    if (mins) mins[id] = lo;
    for (int64_t i = 0; i < g; ++i) {
      const float z = load1(src + i * ld);
      const float q = mm_code(z, lo, inv, levels);
      codes[(gr * g + i) * cols + c] = uint8_t(int(q));
      const float e = __fadd_rn(__fmul_rn(q, s), lo) - z;
      err += e * e;
    }
  }
  if (partial) block_store_partial(err, partial);
}

// The partials in fixed order; sixteen waves with four requests each in flight (four waves with one request each took
// 13.7 us for the 12544 partials of a float32 3584 x 14336 matrix, this takes 5 us).
__global__ __launch_bounds__(1024) void sum_partials_kernel(const double* __restrict__ partial, int n,
                                                            float* __restrict__ out) {
  __shared__ double red[16];
  double t[4] = {0, 0, 0, 0};
  for (int i = threadIdx.x; i < n; i += 4096) {
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] += i + 1024 * u < n ? partial[i + 1024 * u] : 0.0;
  }
  const double w = wave_sum((t[0] + t[1]) + (t[2] + t[3]));
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = w;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0;
    for (int i = 0; i < 16; ++i) s += red[i];
    out[0] = float(s);
  }
}

template <typename Tag, int EPL, int LPG, int U, bool MM>
void launch_col_fast(const RtnArgs& a, float p0, float p1, hipStream_t st, int* nparts) {
  using E = typename Tag::elem;
  const uint32_t nvec = uint32_t(a.rows * a.cols / EPL), colsv = uint32_t(a.cols / EPL);
  const uint32_t nblk = (nvec + kColThreads * U - 1) / (kColThreads * U);
  *nparts = int(nblk);
  if (a.ld == a.cols)
    hipLaunchKernelGGL((rtn_col_fast<Tag, EPL, LPG, U, true, MM>), dim3(nblk), dim3(kColThreads), 0, st, (const E*)a.W, nvec,
                       colsv, a.ld, p0, p1, (uint32_t*)a.codes, a.scales, a.mins, a.partial);
  else
    hipLaunchKernelGGL((rtn_col_fast<Tag, EPL, LPG, U, false, MM>), dim3(nblk), dim3(kColThreads), 0, st, (const E*)a.W, nvec,
                       colsv, a.ld, p0, p1, (uint32_t*)a.codes, a.scales, a.mins, a.partial);
}
// groups of g = 4 .. 256, a power of two, along the contiguous axis
template <typename Tag, bool MM>
void launch_col_groups(const RtnArgs& a, int64_t g, float p0, float p1, hipStream_t st, int* nparts) {
  // bfloat16 in sixteens (g a multiple of 16: so are the rows' lengths, and every piece is 32-byte aligned inside its row)
  if constexpr (Tag::dtype == CAFEQ_BF16) {
    switch (g) {
      case 16: return launch_col_fast<Tag, 16, 1, 2, MM>(a, p0, p1, st, nparts);
      case 32: return launch_col_fast<Tag, 16, 2, 2, MM>(a, p0, p1, st, nparts);
      case 64: return launch_col_fast<Tag, 16, 4, 2, MM>(a, p0, p1, st, nparts);
      case 128: return launch_col_fast<Tag, 16, 8, 2, MM>(a, p0, p1, st, nparts);
      case 256: return launch_col_fast<Tag, 16, 16, 2, MM>(a, p0, p1, st, nparts);
      case 4: return launch_col_fast<Tag, 4, 1, 4, MM>(a, p0, p1, st, nparts);
      default: return launch_col_fast<Tag, 4, 2, 4, MM>(a, p0, p1, st, nparts);
    }
  } else {
    switch (g) {
      case 4: return launch_col_fast<Tag, 4, 1, 4, MM>(a, p0, p1, st, nparts);
      case 8: return launch_col_fast<Tag, 4, 2, 4, MM>(a, p0, p1, st, nparts);
      case 16: return launch_col_fast<Tag, 4, 4, 4, MM>(a, p0, p1, st, nparts);
      case 32: return launch_col_fast<Tag, 4, 8, 4, MM>(a, p0, p1, st, nparts);
      case 64: return launch_col_fast<Tag, 4, 16, 4, MM>(a, p0, p1, st, nparts);
      case 128: return launch_col_fast<Tag, 4, 32, 4, MM>(a, p0, p1, st, nparts);
      default: return launch_col_fast<Tag, 4, 64, 4, MM>(a, p0, p1, st, nparts);
    }
  }
}

// groups of 2048 elements and more that are whole numbers of 16-byte pieces at aligned places and fit the registers of a
// workgroup; false: not such groups
template <typename Tag, bool MM>
bool launch_col_long(const RtnArgs& a, int64_t g, float p0, float p1, hipStream_t st, int* nparts) {
  using E = typename Tag::elem;
  constexpr int PE = Tag::dtype == CAFEQ_BF16 ? 8 : 4;
  if (g < 2048 || g % PE || a.ld % PE || a.cols % PE || g > int64_t(1024) * 16 * PE) return false;
  const int pieces = int(g / PE);
  // eight pieces per lane, or sixteen where even 1024 lanes need them
  int nt = 256;
  while (nt < 1024 && pieces > nt * 8) nt *= 2;
  const int np = (pieces + nt - 1) / nt;
  const int64_t gpr = a.cols / g, ngroups = a.rows * gpr;
  const int nblk = int(std::min<int64_t>(ngroups, 4096));
  *nparts = nblk;
#define CAFEQ_LONG(NP)                                                                                                  \
  hipLaunchKernelGGL((rtn_col_long<Tag, NP, MM>), dim3(nblk), dim3(nt), 0, st, (const E*)a.W, gpr, ngroups, a.cols, a.ld, \
                     int(g), p0, p1, a.codes, a.scales, a.mins, a.partial)
  if (np <= 2) CAFEQ_LONG(2);
  else if (np <= 4) CAFEQ_LONG(4);
  else if (np <= 6) CAFEQ_LONG(6);
  else if (np <= 8) CAFEQ_LONG(8);
  else CAFEQ_LONG(16);
#undef CAFEQ_LONG
  return true;
}

template <typename Tag>
int launch_rtn_typed(const RtnArgs& a, hipStream_t st, int* nparts) {
  using E = typename Tag::elem;
  const int64_t line = a.axis == CAFEQ_AXIS_COL ? a.cols : a.rows;
  const int64_t g = a.group == 0 ? line : a.group;
  *nparts = 0;
  if (a.axis == CAFEQ_AXIS_COL) {
    const bool pow2 = (g & (g - 1)) == 0;
    if (pow2 && g >= 4 && g <= 256 && a.rows * a.cols / 4 < (int64_t(1) << 31)) {
      launch_col_groups<Tag, false>(a, g, a.grid.qmax, a.grid.qmin, st, nparts);
    } else if (!launch_col_long<Tag, false>(a, g, a.grid.qmax, a.grid.qmin, st, nparts)) {
      const int64_t ngroups = a.rows * (a.cols / g);
      const int nblk = int(std::min<int64_t>((ngroups + 3) / 4, 4096));
      *nparts = nblk;
      if (g % 4 == 0 && a.ld % 4 == 0 && a.cols % 4 == 0)
        hipLaunchKernelGGL((rtn_col_vec<Tag>), dim3(nblk), dim3(256), 0, st, (const E*)a.W, a.rows, a.cols,
                           a.ld, g, a.grid, a.codes, a.scales, a.partial);
      else
        hipLaunchKernelGGL((rtn_col_any<Tag>), dim3(nblk), dim3(256), 0, st, (const E*)a.W, a.rows, a.cols,
                           a.ld, g, a.grid, a.codes, a.scales, a.partial);
    }
  } else {
    const int nw = int(g / kRowRPW);
    if (g % kRowRPW == 0 && (nw == 1 || nw == 2 || nw == 4 || nw == 8 || nw == 16) &&
        a.rows / g < 65536) {
      dim3 grid(unsigned((a.cols + 255) / 256), unsigned(a.rows / g));
      *nparts = int(grid.x * grid.y);
#define CAFEQ_ROW_CASE(NW)                                                                          \
  case NW:                                                                                          \
    hipLaunchKernelGGL((rtn_row_fast<Tag, NW>), grid, dim3(NW* kWave), 0, st, (const E*)a.W, a.cols, \
                       a.ld, a.grid, a.codes, a.scales, a.partial);                                 \
    break;
      switch (nw) {
        CAFEQ_ROW_CASE(1)
        CAFEQ_ROW_CASE(2)
        CAFEQ_ROW_CASE(4)
        CAFEQ_ROW_CASE(8)
        CAFEQ_ROW_CASE(16)
      }
#undef CAFEQ_ROW_CASE
    } else {
      const int64_t total = (a.rows / g) * a.cols;
      const int nblk = int(std::min<int64_t>((total + 255) / 256, 4096));
      *nparts = nblk;
      hipLaunchKernelGGL((rtn_row_any<Tag>), dim3(nblk), dim3(256), 0, st, (const E*)a.W, a.rows, a.cols,
                         a.ld, g, a.grid, a.codes, a.scales, a.partial);
    }
  }
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}

template <typename Tag>
int launch_minmax_typed(const RtnArgs& a, float levels, hipStream_t st, int* nparts) {
  using E = typename Tag::elem;
  const int64_t line = a.axis == CAFEQ_AXIS_COL ? a.cols : a.rows;
  const int64_t g = a.group == 0 ? line : a.group;
  if (a.axis == CAFEQ_AXIS_COL) {
    const bool pow2 = (g & (g - 1)) == 0;
    if (pow2 && g >= 4 && g <= 256 && a.rows * a.cols / 4 < (int64_t(1) << 31)) {
      launch_col_groups<Tag, true>(a, g, levels, 0.f, st, nparts);
    } else if (!launch_col_long<Tag, true>(a, g, levels, 0.f, st, nparts)) {
      const int64_t ngroups = a.rows * (a.cols / g);
      const int nblk = int(std::min<int64_t>((ngroups + 3) / 4, 4096));
      *nparts = nblk;
      // load4 needs 16-byte (float32) / 8-byte (bfloat16) aligned groups; the code stores 4-byte aligned ones
      if (g % 4 == 0 && a.ld % 4 == 0 && a.cols % 4 == 0)
        hipLaunchKernelGGL((rtn_col_minmax_vec<Tag>), dim3(nblk), dim3(256), 0, st, (const E*)a.W, a.rows, a.cols,
                           a.ld, g, levels, (uint8_t*)a.codes, a.scales, a.mins, a.partial);
      else
        hipLaunchKernelGGL((rtn_col_minmax_any<Tag>), dim3(nblk), dim3(256), 0, st, (const E*)a.W, a.rows, a.cols,
                           a.ld, g, levels, (uint8_t*)a.codes, a.scales, a.mins, a.partial);
    }
  } else {
    const int64_t total = (a.rows / g) * a.cols;
    const int nblk = int(std::min<int64_t>((total + 255) / 256, 4096));
    *nparts = nblk;
    hipLaunchKernelGGL((rtn_row_minmax_any<Tag>), dim3(nblk), dim3(256), 0, st, (const E*)a.W, a.rows, a.cols,
                       a.ld, g, levels, (uint8_t*)a.codes, a.scales, a.mins, a.partial);
  }
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}

}  // namespace

int launch_rtn_minmax(const RtnArgs& a, int bits, hipStream_t st) {
  int nparts = 0;
  const float levels = float((1 << bits) - 1);
  int rc = a.dtype == CAFEQ_BF16 ? launch_minmax_typed<BF16Tag>(a, levels, st, &nparts)
                                 : launch_minmax_typed<F32Tag>(a, levels, st, &nparts);
  if (rc != CAFEQ_OK) return rc;
  if (a.partial) {
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(1024), 0, st, a.partial, nparts, a.err_sq);
    CAFEQ_CHECK_LAUNCH();
  }
  return CAFEQ_OK;
}

size_t rtn_partials_capacity(int64_t rows, int64_t cols) {
  // upper bound on the number of workgroups any of the four kernels launches
  const int64_t fast = (rows * cols / 4 + kColThreads * kColUnroll - 1) / (kColThreads * kColUnroll);
  const int64_t rowfast = ((cols + 255) / 256) * ((rows + 15) / 16);
  return size_t(std::max<int64_t>(std::max(fast, rowfast), 4096));
}

int launch_rtn(const RtnArgs& a, hipStream_t st) {
  int nparts = 0;
  int rc = a.dtype == CAFEQ_BF16 ? launch_rtn_typed<BF16Tag>(a, st, &nparts)
                                 : launch_rtn_typed<F32Tag>(a, st, &nparts);
  if (rc != CAFEQ_OK) return rc;
  if (a.partial) {
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(1024), 0, st, a.partial, nparts, a.err_sq);
    CAFEQ_CHECK_LAUNCH();
  }
  return CAFEQ_OK;
}

}  // namespace cafeq
