// The loss pass over prepared weights for 32 x 32 transform blocks.
#include "loss_v2.hpp"

namespace cafeq {
int launch_loss_v2_k32(int G, int axis, const CoreParams& p, hipStream_t st) { return launch_v2_k<32>(G, axis, p, st); }
int launch_loss_v2_pair_k32(int G, const CoreParams& pa, const CoreParams& pb, hipStream_t st) { return launch_v2_pair_k<32>(G, pa, pb, st); }
}  // namespace cafeq
