// The loss pass over prepared weights for 64 x 64 transform blocks.
#include "loss_v2.hpp"

namespace cafeq {
int launch_loss_v2_k64(int G, int axis, const CoreParams& p, hipStream_t st) { return launch_v2_k<64>(G, axis, p, st); }
int launch_loss_v2_pair_k64(int G, const CoreParams& pa, const CoreParams& pb, hipStream_t st) { return launch_v2_pair_k<64>(G, pa, pb, st); }
}  // namespace cafeq
