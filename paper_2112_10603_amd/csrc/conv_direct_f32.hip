// fp32 (three-way bf16 split) instantiations of the direct-weight convolution kernel.
#include "conv_direct.h"

namespace ffv {

hipError_t launch_direct_f32(DirectTile tile, const ConvArgs& a, hipStream_t s) {
  using namespace convk;
  const int kind = a.taps == 4 ? 2 : (a.stride == 2 ? 1 : 0);
  switch (tile) {
    case DirectTile::M64N64:
      return kind == 2   ? launch_direct<float, 4, 1, 1, 1, 2, 2, 4, 2>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 1, 1, 2, 2, 6, 2>(a, s)
                         : launch_direct<float, 9, 1, 1, 1, 2, 2, 6, 2>(a, s);
    case DirectTile::M64N128:
      return kind == 2   ? launch_direct<float, 4, 1, 1, 2, 2, 2, 2, 2>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 1, 2, 2, 2, 3, 2>(a, s)
                         : launch_direct<float, 9, 1, 1, 2, 2, 2, 3, 2>(a, s);
    case DirectTile::M128N32:
      return kind == 2   ? launch_direct<float, 4, 1, 1, 1, 4, 1, 4, 2>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 1, 1, 4, 1, 6, 2>(a, s)
                         : launch_direct<float, 9, 1, 1, 1, 4, 1, 6, 2>(a, s);
    case DirectTile::M128N64:
      return kind == 2   ? launch_direct<float, 4, 1, 2, 1, 2, 2, 4, 2>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 2, 1, 2, 2, 6, 2>(a, s)
                         : launch_direct<float, 9, 1, 2, 1, 2, 2, 6, 2>(a, s);
    case DirectTile::M128N128:
      return kind == 2   ? launch_direct<float, 4, 1, 2, 2, 2, 2, 2, 2>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 2, 2, 2, 2, 3, 2>(a, s)
                         : launch_direct<float, 9, 1, 2, 2, 2, 2, 3, 2>(a, s);
    case DirectTile::M32N32K:
      return kind == 2   ? launch_direct<float, 4, 1, 1, 1, 1, 1, 2, 2, kDirectParts>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 1, 1, 1, 1, 3, 2, kDirectParts>(a, s)
                         : launch_direct<float, 9, 1, 1, 1, 1, 1, 3, 2, kDirectParts>(a, s);
    case DirectTile::M64N64F:
      return kind == 2   ? launch_direct<float, 4, 1, 1, 1, 2, 2, 4, 2, 1, true>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 1, 1, 2, 2, 6, 2, 1, true>(a, s)
                         : launch_direct<float, 9, 1, 1, 1, 2, 2, 6, 2, 1, true>(a, s);
    case DirectTile::M64N128F:
      return kind == 2   ? launch_direct<float, 4, 1, 1, 2, 2, 2, 2, 2, 1, true>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 1, 2, 2, 2, 3, 2, 1, true>(a, s)
                         : launch_direct<float, 9, 1, 1, 2, 2, 2, 3, 2, 1, true>(a, s);
    case DirectTile::M128N32F:
      return kind == 2   ? launch_direct<float, 4, 1, 1, 1, 4, 1, 4, 2, 1, true>(a, s)
             : kind == 1 ? launch_direct<float, 9, 2, 1, 1, 4, 1, 6, 2, 1, true>(a, s)
                         : launch_direct<float, 9, 1, 1, 1, 4, 1, 6, 2, 1, true>(a, s);
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace ffv
