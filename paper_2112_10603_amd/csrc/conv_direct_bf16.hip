// bf16 instantiations of the direct-weight convolution kernel.
#include "conv_direct.h"

namespace ffv {

hipError_t launch_direct_bf16(DirectTile tile, const ConvArgs& a, hipStream_t s) {
  using namespace convk;
  const int kind = a.taps == 4 ? 2 : (a.stride == 2 ? 1 : 0);
  switch (tile) {
    case DirectTile::M64N64:
      return kind == 2   ? launch_direct<bf16, 4, 1, 1, 1, 2, 2, 8, 4>(a, s)
             : kind == 1 ? launch_direct<bf16, 9, 2, 1, 1, 2, 2, 18, 4>(a, s)
                         : launch_direct<bf16, 9, 1, 1, 1, 2, 2, 18, 4>(a, s);
    case DirectTile::M128N64:
      return kind == 2   ? launch_direct<bf16, 4, 1, 2, 1, 2, 2, 8, 3>(a, s)
             : kind == 1 ? launch_direct<bf16, 9, 2, 2, 1, 2, 2, 18, 3>(a, s)
                         : launch_direct<bf16, 9, 1, 2, 1, 2, 2, 18, 3>(a, s);
    case DirectTile::M128N128:
      return kind == 2   ? launch_direct<bf16, 4, 1, 2, 2, 2, 2, 8, 2>(a, s)
             : kind == 1 ? launch_direct<bf16, 9, 2, 2, 2, 2, 2, 9, 2>(a, s)
                         : launch_direct<bf16, 9, 1, 2, 2, 2, 2, 9, 2>(a, s);
    case DirectTile::M128N256:  // stride-1 convs only
      return kind == 0 ? launch_direct<bf16, 9, 1, 2, 2, 2, 4, 6, 2>(a, s) : hipErrorInvalidValue;
    case DirectTile::M256N128:  // per-phase transposed convs only
      return kind == 2 ? launch_direct<bf16, 4, 1, 2, 2, 4, 2, 4, 2>(a, s) : hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace ffv
