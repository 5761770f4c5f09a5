// Register-resident Gauss-Jordan inversion of a k x k block by one workgroup: the float64 elimination of the
// blockwise inverse (inverse_kernels.hip: blocks no Newton iteration reaches) and of the adaptive rounding's normal
// equations (adaptive_kernels.hip).
#pragma once
#include <type_traits>

#include "xform_core.hpp"

namespace cafeq {

// Arguments of the Gauss-Jordan inversion (one workgroup per block).
struct GjArgs {
  int K, nz;
  const float* T;        // matrix to invert when partial == nullptr
  const float* partial;  // else [nb][nz][2][K][K]: chunk partials whose first matrix is summed and inverted
  const double* sum64 = nullptr;  // optional with partial: that float64 sum, already formed, [nb][K][K]
  const float* sum32 = nullptr;   // optional with sum64: the same sum rounded to float32 (gj_spd256_kernel reads this)
  float* out;            // [nb][K][K]
  int* status; int status_stride, status_offset;
  // optional [nb][nresid]: shares of a squared residual; a block whose sum is at most resid_max is done (status 0)
  const float* resid = nullptr;
  int nresid = 0;
  float resid_max = 0.f;
};

// Compile-time loop: f(integral_constant<int, I>) for I in [B, E).
template <int B, int E>
struct StaticFor {
  template <typename F>
  static __device__ __forceinline__ void run(F& f) {
    f(std::integral_constant<int, B>{});
    StaticFor<B + 1, E>::run(f);
  }
};
template <int E>
struct StaticFor<E, E> {
  template <typename F>
  static __device__ __forceinline__ void run(F&) {}
};

__device__ __forceinline__ uint32_t dpp_u32_max(uint32_t v, uint32_t o) { return v > o ? v : o; }
// maximum over the wave, returned as a wave-uniform value: DPP inside each row of 16 lanes,
// then the four row results are read back as scalars
__device__ __forceinline__ uint32_t wave_allmax_u32(uint32_t v) {
  v = dpp_u32_max(v, uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0xB1, 0xF, 0xF, true)));    // quad_perm [1,0,3,2]
  v = dpp_u32_max(v, uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x4E, 0xF, 0xF, true)));    // quad_perm [2,3,0,1]
  v = dpp_u32_max(v, uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x141, 0xF, 0xF, true)));   // row_half_mirror
  v = dpp_u32_max(v, uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x140, 0xF, 0xF, true)));   // row_mirror
  const uint32_t a = uint32_t(__builtin_amdgcn_readlane(int(v), 0)), b = uint32_t(__builtin_amdgcn_readlane(int(v), 16));
  const uint32_t c = uint32_t(__builtin_amdgcn_readlane(int(v), 32)), d = uint32_t(__builtin_amdgcn_readlane(int(v), 48));
  return dpp_u32_max(dpp_u32_max(a, b), dpp_u32_max(c, d));
}
// value held by lane `src` (wave-uniform) of a per-lane variable
__device__ __forceinline__ double read_lane(double x, int src) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), src);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), src);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float read_lane(float x, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), src));
}

// |x| as an unsigned key that orders like |x|: the leading 32 bits of the number without its sign
__device__ __forceinline__ uint32_t mag_bits(double x) { return uint32_t(__double2hiint(x)) & 0x7FFFFFFFu; }
__device__ __forceinline__ uint32_t mag_bits(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }

__device__ __forceinline__ double fma_s(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_s(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
// Register-resident in-place Gauss-Jordan inversion with partial pivoting, one workgroup per block.
// Thread (rt, ct) of an NRT x NCT thread grid keeps the RT x CT elements (rt + i*NRT, ct + j*NCT)
// in registers (both strides interleaved, so the LDS reads are either broadcasts or run over
// consecutive addresses).  No physical row swaps: the pivot of column k is the largest entry among
// the rows not yet used (PIV; for symmetric positive definite input, PIV == false, it is the diagonal
// entry), and the pivot order is a permutation undone on output.  One elimination
// step replaces column k by the unit vector e_p and adds multiples of row p / pivot to every row;
// row p itself goes through the same update with the multiplier (1 - pivot), which loses accuracy
// only for |pivot| >> 1, so the block is first scaled by a power of two to max |a_ij| in (1/2, 1].
// The steps of NB = 8 columns (a panel) are taken by the first wave on the K x NB panel alone -- rows
// in registers (lane l holds rows l, l + 64, ...), pivot search by DPP, pivot row through scalar lane
// reads, no barriers -- and their combined effect on the other columns, the rank-NB update
// R += C . X  (C: the panel after its steps minus the unit vectors of the pivot rows, X: the NB pivot
// rows as they were before the panel), is applied by all threads at once: three barriers per panel.
// A singular block keeps running (on infinities) and is zeroed at the end.
//   A = T_b (float32) when partial == nullptr, else the float64 sum over nz chunk partials
//   of S (first of the two K x K matrices of each partial).  out = A^-1 (zeros if singular).
template <int K, typename S>
struct GjShared {
  static constexpr int NB = 8;
  S pan[2][K][NB];
  S xrow[2][NB][K];
  S wred[16];
  int pk[K], kinv[K];
  int pvt[2][NB];
  int deadflag;
};
// (K / RT) * (K / CT) threads; sh: 16-byte aligned LDS
template <int K, int RT, int CT, typename S, bool PIV>
__device__ void gj_panel_body(const GjArgs& a, const int b, GjShared<K, S>& sh) {
  constexpr int NRT = K / RT, NCT = K / CT, NTHR = NRT * NCT, NWAVE = (NTHR + 63) / 64;
  constexpr int NB = 8, NPH = NCT / NB, NRW = (K + 63) / 64;
  static_assert(NCT % NB == 0, "panel width");
  auto& pan = sh.pan;
  auto& xrow = sh.xrow;
  auto& wred = sh.wred;
  auto& pk = sh.pk;
  auto& kinv = sh.kinv;
  auto& pvt = sh.pvt;
  auto& deadflag = sh.deadflag;
  const int tid = threadIdx.x, lane = tid & 63;
  const int rt = tid / NCT, ct = tid % NCT;
  S reg[RT][CT];
  if (a.partial == nullptr) {
    const float* src = a.T + size_t(b) * K * K;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) reg[i][j] = S(src[(rt + i * NRT) * K + ct + j * NCT]);
  } else if (a.sum64) {
    // one workgroup reading nz partials of its block is a long serial prologue when the blocks are few:
    // the float64 sum then comes from a kernel that spreads that work over the chip
    const double* src = a.sum64 + size_t(b) * K * K;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) reg[i][j] = S(src[(rt + i * NRT) * K + ct + j * NCT]);
  } else {
    const float* src = a.partial + size_t(b) * a.nz * 2 * K * K;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) reg[i][j] = 0;
    for (int z = 0; z < a.nz; ++z) {
      // float64 accumulation; the float elimination (K = 256) rounds the sum once
      double t[RT][CT];
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) t[i][j] = double(src[size_t(z) * 2 * K * K + (rt + i * NRT) * K + ct + j * NCT]);
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) reg[i][j] = S(double(reg[i][j]) + t[i][j]);
    }
  }
  S anorm = 0;
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) anorm = fmax(anorm, fabs(reg[i][j]));
  for (int m = 1; m < 64; m <<= 1) anorm = fmax(anorm, __shfl_xor(anorm, m));
  if (lane == 0) wred[tid >> 6] = anorm;
  if (tid == 0) deadflag = 0;
  __syncthreads();
  anorm = 0;
  for (int i = 0; i < NWAVE; ++i) anorm = fmax(anorm, wred[i]);
  int ex = 0;
  (void)frexp(double(anorm), &ex);
  const S scale = S(ldexp(1.0, -ex));    // exact power of two; 1 if the block is all zero
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) reg[i][j] *= scale;
  const S tol = anorm * scale * S(a.partial ? 1e-5 : (sizeof(S) == 8 ? 1e-12 : 1e-6));
  uint32_t usedbits = 0;   // first wave only: bit q = row lane + 64 q has been a pivot

  auto panels = [&](auto jj_c) {
    constexpr int jj = decltype(jj_c)::value;
    for (int h = 0; h < NPH; ++h) {
      const int buf = (jj * NPH + h) & 1;
      const int q_own = ct - h * NB;
      const bool owner = q_own >= 0 && q_own < NB;
      if (owner) {
#pragma unroll
        for (int i = 0; i < RT; ++i) pan[buf][rt + i * NRT][q_own] = reg[i][jj];
      }
      __syncthreads();
      if (tid < 64) {
        S prow[NRW][NB];
#pragma unroll
        for (int q = 0; q < NRW; ++q) {
          const int rr = lane + 64 * q;
#pragma unroll
          for (int c = 0; c < NB; ++c) prow[q][c] = rr < K ? pan[buf][rr < K ? rr : 0][c] : S(0);
        }
        int pivs[NB];
        bool dd = false;
#pragma unroll
        for (int s = 0; s < NB; ++s) {
          // pivot = (approximately) largest |entry| of the column among the unused rows: a 32-bit key
          // (leading bits of the magnitude, low byte 255 - row: ties go to the lowest row) reduced by DPP
          // (PIV == false, for symmetric positive definite input: the diagonal entry, no search)
          S colv[NRW];
          uint32_t key = 0x100u;
#pragma unroll
          for (int q = 0; q < NRW; ++q) colv[q] = prow[q][s];
          int p = jj * NCT + h * NB + s;
          if (PIV) {
            key = 0;
#pragma unroll
            for (int q = 0; q < NRW; ++q) {
              const int rr = lane + 64 * q;
              const uint32_t kk_ = (rr >= K || ((usedbits >> q) & 1u)) ? 0u
                                                                       : ((mag_bits(colv[q]) & 0xFFFFFF00u) | uint32_t(255 - rr));
              key = key > kk_ ? key : kk_;
            }
            key = wave_allmax_u32(key);
            p = (255 - int(key & 0xFFu)) & (K - 1);
          }
          const int pl = p & 63, pq = p >> 6;
          S pv = read_lane(colv[0], pl);
#pragma unroll
          for (int q = 1; q < NRW; ++q) {
            const S alt = read_lane(colv[q], pl);
            pv = pq == q ? alt : pv;
          }
          dd = dd || (key >> 8) == 0 || !((PIV ? S(fabs(pv)) : pv) > tol);
          // reciprocal of the pivot: hardware estimate (2^-22) + Newton steps to full precision
          S ipiv = S(__builtin_amdgcn_rcpf(float(pv)));
          ipiv = ipiv * (S(2) - pv * ipiv);
          if (sizeof(S) == 8) ipiv = ipiv * (S(2) - pv * ipiv);
          // row p of the panel, with the in-place 1 in the column of this step
          S rowp[NB];
#pragma unroll
          for (int c = 0; c < NB; ++c) {
            S mine = prow[0][c];
#pragma unroll
            for (int q = 1; q < NRW; ++q) mine = pq == q ? prow[q][c] : mine;
            rowp[c] = c == s ? S(1) : read_lane(mine, pl);
          }
#pragma unroll
          for (int q = 0; q < NRW; ++q) {
            const bool isp = (lane + 64 * q) == p;
            const S f = (isp ? S(1) - pv : -colv[q]) * ipiv;
#pragma unroll
            for (int c = 0; c < NB; ++c)
              prow[q][c] = c == s ? (isp ? S(1) : S(0)) + f : fma_s(f, rowp[c], prow[q][c]);
            usedbits |= uint32_t(isp) << q;
          }
          pivs[s] = p;
        }
        // hand over C = (panel after its steps) - (unit vectors of the pivot rows), and the pivots
#pragma unroll
        for (int q = 0; q < NRW; ++q) {
          const int rr = lane + 64 * q;
          if (rr < K) {
#pragma unroll
            for (int c = 0; c < NB; ++c) pan[buf][rr][c] = prow[q][c] - (rr == pivs[c] ? S(1) : S(0));
          }
        }
        if (lane == 0) {
#pragma unroll
          for (int c = 0; c < NB; ++c) {
            pvt[buf][c] = pivs[c];
            pk[jj * NCT + h * NB + c] = pivs[c];
          }
          if (dd) deadflag = 1;
        }
      }
      __syncthreads();
      // the owners of the pivot rows publish them as they were before the panel
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const int p = pvt[buf][c];
        const int prt = p % NRT;
        if constexpr (!PIV && NRT % NCT == 0) {
          // diagonal pivots p = jj NCT + h NB + c: the register row p / NRT does not depend on h and c
          constexpr int pi = (jj * NCT) / NRT;
          if (rt == prt) {
#pragma unroll
            for (int j = 0; j < CT; ++j) xrow[buf][c][ct + j * NCT] = reg[pi][j];
          }
        } else {
          // (one flat condition per register row: nesting the row test inside the thread test made the
          // compiler index the registers dynamically, through scratch memory)
          const int pi = p / NRT;
#pragma unroll
          for (int i = 0; i < RT; ++i)
            if (rt == prt && i == pi) {
#pragma unroll
              for (int j = 0; j < CT; ++j) xrow[buf][c][ct + j * NCT] = reg[i][j];
            }
        }
      }
      __syncthreads();
#pragma unroll 2
      for (int c = 0; c < NB; ++c) {
        S xv[CT], cr[RT];
#pragma unroll
        for (int j = 0; j < CT; ++j) xv[j] = xrow[buf][c][ct + j * NCT];
#pragma unroll
        for (int i = 0; i < RT; ++i) cr[i] = pan[buf][rt + i * NRT][c];
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < CT; ++j) reg[i][j] = fma_s(cr[i], xv[j], reg[i][j]);
      }
      // a panel column becomes the panel's own result
      if (owner) {
        const int pq = pvt[buf][q_own];
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const int r = rt + i * NRT;
          reg[i][jj] = pan[buf][r][q_own] + (r == pq ? S(1) : S(0));
        }
      }
    }
  };
  StaticFor<0, CT>::run(panels);
  __syncthreads();
  const bool dead = deadflag != 0;
  if (a.status && tid == 0) a.status[size_t(b) * a.status_stride + a.status_offset] = dead ? 1 : 0;
  float* O = a.out + size_t(b) * K * K;
  if (dead) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) O[(rt + i * NRT) * K + ct + j * NCT] = 0.f;
    return;
  }
  if (tid < K) kinv[pk[tid]] = tid;
  __syncthreads();
  // register (r, c) is element (kinv[r], pk[c]) of the inverse of the scaled block
  int ocol[CT];
#pragma unroll
  for (int j = 0; j < CT; ++j) ocol[j] = pk[ct + j * NCT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int orow = kinv[rt + i * NRT];
#pragma unroll
    for (int j = 0; j < CT; ++j) O[orow * K + ocol[j]] = float(reg[i][j] * scale);
  }
}
template <int K, int RT, int CT, typename S, bool PIV>
__global__ __launch_bounds__((K / RT) * (K / CT)) void gj_panel_kernel(const GjArgs a) {
  __shared__ __align__(16) GjShared<K, S> sh;
  if (a.resid) {
    float t = 0.f;
    for (int q = 0; q < a.nresid; ++q) t += a.resid[size_t(blockIdx.x) * a.nresid + q];
    if (t <= a.resid_max) {                        // uniform over the workgroup (a NaN is not done)
      if (a.status && threadIdx.x == 0) a.status[size_t(blockIdx.x) * a.status_stride + a.status_offset] = 0;
      return;
    }
  }
  gj_panel_body<K, RT, CT, S, PIV>(a, int(blockIdx.x), sh);
}

}  // namespace cafeq
