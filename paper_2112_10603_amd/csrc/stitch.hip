// Multi-view cluster frame (the paper's Multiview Organizer, section 3.2,
// and the supplement's 16-views-per-side clusters): a camera's real view at
// full resolution between two blocks of its neighbouring views, each
// downscaled by g in both directions (g x g box mean) and tiled g x g in
// raster order, so a side's g*g views fill exactly one H x W block:
//   frame [3][H][3W] = [left block | real view | right block].
// Memory-bound (2 g^2 + 1 views read, 3 written). strip4_k, for g = 4 with
// tiles at least 64 pixels wide: a workgroup takes one output row of one view
// and plane, i.e. four whole source rows, which lie together in memory, and
// reads and writes past the caches (nothing is used twice). stitch_k: one
// thread per output pixel in frame order, where a workgroup's pixels come
// from several views; the other g keep it (g = 1, 2 and 8 measured 1 to 9 %
// faster with it than in uncached strips), as does g = 4 with a real view or a
// frame that is not 16-byte aligned (its side views always are: both kernels
// read them in 16-byte loads, and the entry point refuses others).
// 1080 x 1920, g = 4 (896 MB): 177 -> 161 us (5.6 TB/s); cached loads in the
// same strips take 172 us, two strips per workgroup 160.
#include "common.h"

namespace ffv {

namespace {

constexpr int TPB = 256;

template <int G>
__global__ void stitch_k(StitchArgs a) {
  const long HW3 = 3L * a.H * a.W;  // pixels of one output plane
  const long p = (long)blockIdx.x * TPB + threadIdx.x;
  if (p >= HW3) return;
  const int W3 = 3 * a.W;
  const int y = (int)(p / W3), x = (int)(p % W3);
  const int block = x / a.W, xl = x - block * a.W;
  const long HWs = (long)a.H * a.W;
  float v[3];
  if (block == 1) {
    const long q = (long)y * a.W + xl;
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = a.hr[c * HWs + q];
  } else {
    const int th = a.H / G, tw = a.W / G;
    const int r = y / th, qd = xl / tw;
    const float* src = a.views[(block == 0 ? 0 : a.n) + r * G + qd];
    const int sy = G * (y - r * th), sx = G * (xl - qd * tw);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float* s = src + c * HWs + (long)sy * a.W + sx;
      float acc = 0.f;
#pragma unroll
      for (int i = 0; i < G; ++i) {
        if constexpr (G == 4) {
          const float4 t = *reinterpret_cast<const float4*>(s + (long)i * a.W);
          acc += (t.x + t.y) + (t.z + t.w);
        } else {
#pragma unroll
          for (int j = 0; j < G; ++j) acc += s[(long)i * a.W + j];
        }
      }
      v[c] = acc * (1.f / (G * G));
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) a.out[c * HW3 + p] = v[c];
}

// g = 4. Workgroups [0, sides): output row y of plane c of side view vi; the
// rest: a row of a plane of the real view. Every pointer is 16-byte aligned.
__global__ __launch_bounds__(TPB) void strip4_k(StitchArgs a, int sides) {
  const long HW3 = 3L * a.H * a.W, HWs = (long)a.H * a.W;
  const int W3 = 3 * a.W;
  const int th = a.H / 4, tw = a.W / 4;
  int b = blockIdx.x;
  if (b >= sides) {
    b -= sides;
    const int c = b / a.H, y = b - c * a.H;
    const f32x4* s = reinterpret_cast<const f32x4*>(a.hr + c * HWs + (long)y * a.W);
    f32x4* o = reinterpret_cast<f32x4*>(a.out + c * HW3 + (long)y * W3 + a.W);
    for (int x = threadIdx.x; x < tw; x += TPB) __builtin_nontemporal_store(__builtin_nontemporal_load(s + x), o + x);
    return;
  }
  const int y = b % th;
  b /= th;
  const int c = b % 3, vi = b / 3;
  const int side = vi >= a.n ? 1 : 0, k = vi - side * a.n;
  const float* s = a.views[vi] + c * HWs + 4L * y * a.W;
  float* o = a.out + c * HW3 + (long)((k >> 2) * th + y) * W3 + 2 * side * a.W + (k & 3) * tw;
  for (int x = threadIdx.x; x < tw; x += TPB) {
    f32x4 t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      t[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(s + (long)i * a.W + 4 * x));
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc += (t[i].x + t[i].y) + (t[i].z + t[i].w);
    __builtin_nontemporal_store(acc * (1.f / 16), o + x);
  }
}

template <int G>
hipError_t launch_g(const StitchArgs& a, hipStream_t s) {
  if constexpr (G == 4) {
    const uintptr_t bits = reinterpret_cast<uintptr_t>(a.hr) | reinterpret_cast<uintptr_t>(a.out);
    const long sides = 2L * a.n * 3 * (a.H / 4), blocks = sides + 3L * a.H;
    if (bits % 16 == 0 && a.W / 4 >= 64 && blocks <= 0x7fffffffL) {
      hipLaunchKernelGGL(strip4_k, dim3((unsigned)blocks), dim3(TPB), 0, s, a, (int)sides);
      return hipGetLastError();
    }
  }
  const long n = 3L * a.H * a.W;
  hipLaunchKernelGGL(stitch_k<G>, dim3((unsigned)((n + TPB - 1) / TPB)), dim3(TPB), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_stitch(const StitchArgs& a, hipStream_t s) {
  if (a.H <= 0 || a.W <= 0) return hipSuccess;
  switch (a.g) {
    case 1: return launch_g<1>(a, s);
    case 2: return launch_g<2>(a, s);
    case 4: return launch_g<4>(a, s);
    case 8: return launch_g<8>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ffv
