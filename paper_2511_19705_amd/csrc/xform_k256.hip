// Instantiations of the fused transform core for 256 x 256 transform blocks: groups of several blocks.  Groups inside a block
// go through xform256.hip.
#include "xform_launch.hpp"
namespace cafeq {
int launch_core_k256(int G, int axis, const CoreParams& p, hipStream_t st) {
  if (!p.longg) return launch_xform256(G, axis, p, st);
  if (G != 256 || p.do_grad || p.fscale) return CAFEQ_ERR_INVALID_ARG;
  const size_t lds = core_lds_bytes_t<256, 256>(false);
  if (p.sweep)
    return axis == CAFEQ_AXIS_COL ? launch_sweep<256, 256, CAFEQ_AXIS_COL, false>(p, lds, st)
                                  : launch_sweep<256, 256, CAFEQ_AXIS_ROW, false>(p, lds, st);
  return axis == CAFEQ_AXIS_COL ? launch_core_v<256, 256, CAFEQ_AXIS_COL, false, false, true>(p, lds, st)
                                : launch_core_v<256, 256, CAFEQ_AXIS_ROW, false, false, true>(p, lds, st);
}
size_t core_lds_bytes_k256(int G, bool do_grad) { return core_lds_bytes_k<256>(G, do_grad); }
}  // namespace cafeq
