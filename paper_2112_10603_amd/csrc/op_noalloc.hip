// ffv_op_conv_noalloc: the op-level convolution with its device buffers in
// a fixed per-device array instead of hipMalloc'd memory, for callers that
// cannot allocate.
#include <mutex>

#include <hip/hip_runtime.h>

#include "../../include/ffv.h"
#include "op_conv.h"

namespace {

// Scratch of every ffv_op_conv_noalloc call on a device: the NHWC input
// copy, packed weights, bias, NHWC output and zero block. Each device holds
// its own copy, at its own address, until the process ends.
constexpr size_t kScratchBytes = (size_t)FFV_OP_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
// Weights of the direct-weight kernel: apart, so that the layers that fit the
// array do not depend on the kernel that runs them.
static __device__ __align__(256) unsigned char direct_weights[ffv::kOpDirectBytes];

constexpr int kMaxDevices = 64;
std::mutex g_mu;
struct Arrays {
  void *scratch, *direct;
};
Arrays g_ptr[kMaxDevices] = {};  // their device addresses, per device

}  // namespace

extern "C" ffv_status ffv_op_conv_noalloc(int32_t precision, const float* x, int32_t n, int32_t cin,
                                          int32_t h, int32_t w, const float* weight, const float* bias,
                                          int32_t cout, int32_t stride, int32_t transposed, int32_t relu,
                                          int32_t n_tile, int32_t tile_w, float* y, void* stream) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return ffv::op_fail(FFV_ERR_DEVICE, "no current HIP device");
  Arrays at{};
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_ptr[dev].scratch) {
      // first call on this device (which is current): the arrays' device
      // addresses; host code never uses the arrays' own names
      hipError_t e = hipGetSymbolAddress(&at.scratch, HIP_SYMBOL(scratch));
      if (e == hipSuccess) e = hipGetSymbolAddress(&at.direct, HIP_SYMBOL(direct_weights));
      if (e != hipSuccess || !at.scratch || !at.direct) return ffv::op_fail(FFV_ERR_DEVICE, hipGetErrorString(e));
      g_ptr[dev] = at;
    }
    at = g_ptr[dev];
  }
  const ffv::OpConvScratch sc{at.scratch, kScratchBytes, at.direct};
  return ffv::op_conv_run(&sc, precision, x, n, cin, h, w, weight, bias, cout, stride, transposed, relu,
                          n_tile, tile_w, y, stream);
}
