// fp8 instantiations of the direct-weight convolution kernel.
#include "conv_direct.h"

namespace ffv {

hipError_t launch_direct_f8(DirectTile tile, const ConvArgs& a, hipStream_t s) {
  using namespace convk;
  const int kind = a.taps == 4 ? 2 : (a.stride == 2 ? 1 : 0);
  switch (tile) {
    case DirectTile::M64N64:
      return kind == 2   ? launch_direct<f8, 4, 1, 1, 1, 2, 2, 4, 2>(a, s)
             : kind == 1 ? launch_direct<f8, 9, 2, 1, 1, 2, 2, 9, 2>(a, s)
                         : launch_direct<f8, 9, 1, 1, 1, 2, 2, 9, 2>(a, s);
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace ffv
