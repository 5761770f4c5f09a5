// Blockwise inverse of the transform for blocks of 32, 64 and 128 (S0 of the path; blocks of 256: adaptive_kernels.hip).
//
// The transforms of this method stay near scaled rotations: they start as rotations and gradient steps move them a
// little at a time.  So a block is first tried with Newton's iteration  X <- X + X R,  R = I - T X  (R_new = R^2),
// from X0 = T^T / alpha, alpha = ||T||_F^2 / k, the exact inverse of a rotation scaled by any factor, or from the
// inverse of the loop's previous iteration.  The residual is measured in every round, and the iteration's result is
// used only where the residual it reached is small; any other block -- no convergence, overflow, singular -- goes
// through the float64 elimination of gj_panel.hpp inside the same launch.
//
// Why products instead of the elimination: the elimination is a serial chain of k pivot steps (0.75 us each at
// k = 128), while a round is two k x k products on the 16-bit matrix pipe: 9.3 k cycles at k = 128, of which 3.7 k are
// the products and the rest splitting, LDS and barriers.  Measured, blocks 5 % off rotations, against a launch that
// checked for rotations and one that eliminated the others: 112 blocks of 128 11 + 111 -> 31 us (57 k cycles: start 14 k,
// three rounds 28 k, the exact step 15 k), 288 blocks (more than one per compute unit) 26 + 198 -> 60 us, 144 blocks of
// 64 5 + 36 -> 11.5 us, 8 blocks of 32 16.6 -> 7.5 us; the learning loops' warm start at 72 blocks of 128 30 + 5 -> 23.5 us.
// A block that Newton does not reach pays its rounds: whole calls on blocks far from rotations 16.6 -> 17.7 us for 8 blocks of
// 32 (up to 25 where a few of many give up late, 20 to 30 % off), 95.7 -> 99.8 us for 8 and 102.2 -> 103.3 us for 112 of 128.
#include <atomic>

#include "ns_inverse.hpp"

namespace cafeq {
namespace {

template <int K, int WARM>
__global__ __launch_bounds__(NsShape<K>::NW * 64) void ns_inverse_kernel(const float* __restrict__ T, float* __restrict__ Tinv,
                                                                         int* __restrict__ status) {
  extern __shared__ __align__(16) unsigned char ns_lds[];
  const int b = int(blockIdx.x);
  if (!ns_inverse_body<K, WARM>(T, Tinv, status, b, ns_lds))
    gj_panel_body<K, 4, 4 * NsShape<K>::TPW, double, true>(ns_eliminate_args(K, T, Tinv, status), b, *reinterpret_cast<GjShared<K, double>*>(ns_lds));
}

template <int K, int WARM>
int launch_ns(const float* T, int nb, float* Tinv, int* status, hipStream_t st) {
  constexpr size_t lds = NsShape<K>::bytes;
  if (lds > 64 * 1024) {
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(ns_inverse_kernel<K, WARM>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)
        return CAFEQ_ERR_LAUNCH;
      attr_set = true;
    }
  }
  hipLaunchKernelGGL((ns_inverse_kernel<K, WARM>), dim3(nb), dim3(NsShape<K>::NW * 64), lds, st, T, Tinv, status);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}
}  // namespace

int launch_block_inverse(const float* T, int K, int nb, double* work, float* Tinv, float* rho_row, float* rho_col,
                         int* status, hipStream_t st) {
  int rc = CAFEQ_ERR_UNSUPPORTED;
  switch (K) {
    case 32: rc = launch_ns<32, 0>(T, nb, Tinv, status, st); break;
    case 64: rc = launch_ns<64, 0>(T, nb, Tinv, status, st); break;
    case 128: rc = launch_ns<128, 0>(T, nb, Tinv, status, st); break;
    case 256: return launch_inverse256(T, nb, work, Tinv, rho_row, rho_col, status, false, st);
  }
  if (rc) return rc;
  RhoRequest rho[2];
  int nrho = 0;
  if (rho_row) rho[nrho++] = RhoRequest{Tinv, rho_row, 1};
  if (rho_col) rho[nrho++] = RhoRequest{Tinv, rho_col, 0};
  if (nrho && (rc = launch_split_planes_multi(nullptr, 0, K, nb, st, nullptr, 0, rho, nrho))) return rc;
  return CAFEQ_OK;
}

// The inverse inside a learning loop: Tinv holds the previous iteration's inverse on entry.
int launch_block_inverse_warm(const float* T, int K, int nb, double* work, float* Tinv, int* status, hipStream_t st) {
  switch (K) {
    case 32: return launch_ns<32, 1>(T, nb, Tinv, status, st);
    case 64: return launch_ns<64, 1>(T, nb, Tinv, status, st);
    case 128: return launch_ns<128, 1>(T, nb, Tinv, status, st);
    case 256: return launch_inverse256(T, nb, work, Tinv, nullptr, nullptr, status, true, st);
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
}

}  // namespace cafeq
