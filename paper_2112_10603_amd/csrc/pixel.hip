// Per-pixel passes of the view-interpolation network: ingest and padding,
// the image pyramid, stage input assembly with flow upscaling and backward
// warps (Eq. 2), the final warp and mask blend (Eq. 1), the flow pyramid and
// the context-feature warps of the refinement U-Net, and the output head.
//
// All are memory-bound: one thread per output pixel (or per 8-channel group
// of a pixel), NHWC so the threads of a wavefront touch consecutive pixels.
// Sample positions, bilinear weights, flows and the mask stay fp32 in every
// precision; only the activations fed to convolutions use the activation
// dtype.
#include <type_traits>

#include "common.h"

namespace ffv {

namespace {

constexpr int TPB = 256;

template <typename T>
__device__ inline T cvt(float v) {
  return (T)v;
}

__device__ inline float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// 16-byte packing of activation values: N values (N a multiple of 8 for
// bf16, of 4 for fp32) written to dst with 16-byte stores (dst 16-byte
// aligned), and 8 values read back with one or two 16-byte loads.
__device__ inline uint32_t pack2(float a, float b) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (bf16)a) | ((uint32_t)__builtin_bit_cast(uint16_t, (bf16)b) << 16);
}

template <typename T, int N>
__device__ inline void store_vals(T* dst, const float (&v)[N]) {
  if constexpr (sizeof(T) == 2) {
    static_assert(N % 8 == 0, "whole 16-byte chunks");
#pragma unroll
    for (int k = 0; k < N; k += 8)
      *reinterpret_cast<uint4*>(dst + k) =
          make_uint4(pack2(v[k], v[k + 1]), pack2(v[k + 2], v[k + 3]), pack2(v[k + 4], v[k + 5]),
                     pack2(v[k + 6], v[k + 7]));
  } else {
    static_assert(N % 4 == 0, "whole 16-byte chunks");
#pragma unroll
    for (int k = 0; k < N; k += 4)
      *reinterpret_cast<float4*>(dst + k) = make_float4(v[k], v[k + 1], v[k + 2], v[k + 3]);
  }
}

// N values as 16-byte chunks in the layout store_vals writes.
template <typename T, int N>
__device__ inline void pack_chunks(const float (&v)[N], uint4 (&c)[N * sizeof(T) / 16]) {
  if constexpr (sizeof(T) == 2) {
    static_assert(N % 8 == 0, "whole 16-byte chunks");
#pragma unroll
    for (int k = 0; k < N; k += 8)
      c[k / 8] = make_uint4(pack2(v[k], v[k + 1]), pack2(v[k + 2], v[k + 3]), pack2(v[k + 4], v[k + 5]),
                            pack2(v[k + 6], v[k + 7]));
  } else {
    static_assert(N % 4 == 0, "whole 16-byte chunks");
#pragma unroll
    for (int k = 0; k < N; k += 4)
      c[k / 4] = make_uint4(__float_as_uint(v[k]), __float_as_uint(v[k + 1]), __float_as_uint(v[k + 2]),
                            __float_as_uint(v[k + 3]));
  }
}

// Wave-contiguous stores of per-pixel records through LDS. The 64 lanes of a
// wave hold the NC-chunk records of 64 consecutive pixels, contiguous in
// memory. Stored lane by lane, each store instruction covers one chunk in NC
// of the wave's span, so every line is written in NC partial pieces and the
// write requests multiply by NC (measured: the 48-byte records of the stage
// transition took 5.5 of its 8.6 ms at 1080p x 112 views). Instead each lane
// puts its record into the wave's LDS area (stage_put) and, a wave's LDS
// accesses being in order (wave_sync holds the compiler to it), each store
// instruction then writes 64 consecutive chunks (stage_flush); records of
// pixels at or past the row's last one are not written. These stores, and the final pass's blended image, are marked
// non-temporal: a pass streams out far more than the caches hold, so
// keeping its output lines cached only evicts the camera rows and flow
// taps its waves are still gathering (measured at 1080p x 112 views: final
// pass 8.96 -> 8.38 ms, stage transitions 9.04 -> 8.71 ms, the kernels
// that read the records unchanged).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ inline void store_nt(uint4* dst, const uint4& w) {
  const u32x4 v = {w.x, w.y, w.z, w.w};
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
}

__device__ inline void store_nt(float* dst, const float4& w) {
  const f32x4 v = {w.x, w.y, w.z, w.w};
  __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(dst));
}

__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int NC>
__device__ inline void stage_put(uint4* wave_stage, int lane, const uint4 (&c)[NC]) {
#pragma unroll
  for (int k = 0; k < NC; ++k) wave_stage[lane * NC + k] = c[k];
}

template <int NC>
__device__ inline void stage_flush(const uint4* wave_stage, int lane, uint4* dst, int n_valid) {
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int c = k * 64 + lane;
    if (c / NC < n_valid) store_nt(dst + c, wave_stage[c]);
  }
}

template <typename T>
__device__ inline void load8(const T* src, float (&v)[8]) {
  if constexpr (sizeof(T) == 2) {
    const uint4 u = *reinterpret_cast<const uint4*>(src);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[2 * k] = __uint_as_float(w[k] << 16);
      v[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
    }
  } else {
    const float4 a = *reinterpret_cast<const float4*>(src), b = *reinterpret_cast<const float4*>(src + 4);
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
  }
}

// Workgroups of the passes that warp full images take 64 x 4 pixel tiles (a
// wave a row of 64): the bilinear taps of a tile's rows overlap, and where
// the flow is rough they scatter over neighbouring rows, which a tile keeps
// in its L1 and a run of one row does not. Consecutive workgroup ids go to
// the 8 XCDs in turn, each with its own L2, so an XCD takes columns of
// kSuper tiles one above the other, the XCDs side by side in the same image
// rows. views_fast: a column's tile in every view before the next tile, so
// that views of one camera pair share its rows in the L2; otherwise view
// after view, which keeps fewer output streams open at a time. Smooth flow /
// flow with 4 pixels of noise, us, rows of 256 pixels -> tiles: final pass of
// 4 views of 4K 827 -> 764 / 1427 -> 1022 (128 bytes a pixel: 5.6 / 4.2
// TB/s), 24 of 1080p 1147 -> 1074 / 1635 -> 1382, one of 720p 18.5 -> 19.8 /
// 23.5 -> 21.5; stage transition of 4 views of 4K 940 -> 869 / 1114 -> 959, 3
// of 1080p 137 -> 91 / 161 -> 100, one of 720p 28 -> 19.5 / 33 -> 20.
constexpr int kSuper = 8;
inline dim3 super_grid(int h, int w, int n_views, bool views_fast) {
  const long cols = (w + 63) / 64, sup = cols * (((h + 3) / 4 + kSuper - 1) / kSuper);
  const unsigned sup8 = (unsigned)((sup + 7) / 8), n = (unsigned)n_views;
  return views_fast ? dim3(8 * n, kSuper, sup8) : dim3(8 * kSuper, sup8, n);
}
// The tile (x, y) and view of this workgroup in a launch of images w wide.
__device__ inline void super_tile(int w, bool views_fast, int& tx, int& ty, int& v) {
  const int q = blockIdx.x >> 3, cols = (w + 63) / 64;
  v = views_fast ? q : (int)blockIdx.z;
  const unsigned sup = (views_fast ? blockIdx.z : blockIdx.y) * 8 + (blockIdx.x & 7), sy = sup / (unsigned)cols;
  tx = (int)(sup - sy * cols);
  ty = (int)(sy * kSuper) + (views_fast ? (int)blockIdx.y : q);
}

// Workgroup order within one image of a (pixel blocks x images) grid, for
// passes that read a pixel's neighbours (3x3 taps, bilinear warp and
// upsampling taps). Consecutive workgroup ids go to the 8 XCDs in turn,
// each with its own L2, so in launch order the block below a block (one
// row of 1920 pixels is 7.5 blocks) runs on another XCD and every row is
// fetched into several L2s. Here the blocks that land on one XCD take a
// contiguous band of the image instead, while all XCDs still work on the
// same image at the same time (its cameras' rows stay shared in the
// last-level cache). Measured at 1080p x 112 views: L2 misses of the
// context warps fall 3.3x and of the head 2.1x, for 5-15 % and 2 % less
// time (these passes wait on latency more than on bytes). (The context warps
// in tiles four rows high measured 2 to 10 % slower than in this order.)
__device__ inline long banded(unsigned i, unsigned gx) {  // block i of gx
  // the blocks of this image with the same id mod 8 share an XCD
  const unsigned r = i & 7u, q = gx >> 3, rem = gx & 7u;
  return (long)(r * q + (r < rem ? r : rem) + (i >> 3));
}
__device__ inline long banded_block() { return banded(blockIdx.x, gridDim.x); }

// Half-pixel-centre source coordinate for resampling n_in -> n_out.
__device__ inline void hp_tap(int i, int n_in, int n_out, int& i0, int& i1, float& w) {
  float s = ((float)i + 0.5f) * ((float)n_in / (float)n_out) - 0.5f;
  s = fmaxf(s, 0.f);
  int f = (int)floorf(s);
  if (f > n_in - 1) f = n_in - 1;
  i0 = f;
  i1 = min(f + 1, n_in - 1);
  w = s - (float)f;
}

// Backward bilinear sample position u + f, clamped to the image (border mode).
struct Tap4 {
  int o00, o01, o10, o11;  // pixel offsets
  float w00, w01, w10, w11;
};

__device__ inline Tap4 warp_taps(int x, int y, float fx, float fy, int w, int h) {
  float px = fminf(fmaxf((float)x + fx, 0.f), (float)(w - 1));
  float py = fminf(fmaxf((float)y + fy, 0.f), (float)(h - 1));
  int x0 = (int)floorf(px), y0 = (int)floorf(py);
  int x1 = min(x0 + 1, w - 1), y1 = min(y0 + 1, h - 1);
  float a = px - (float)x0, b = py - (float)y0;
  Tap4 t;
  t.o00 = y0 * w + x0;
  t.o01 = y0 * w + x1;
  t.o10 = y1 * w + x0;
  t.o11 = y1 * w + x1;
  t.w00 = (1.f - a) * (1.f - b);
  t.w01 = a * (1.f - b);
  t.w10 = (1.f - a) * b;
  t.w11 = a * b;
  return t;
}

__device__ inline float4 sample4(const float* img, const Tap4& t) {
  float4 p00 = ld4(img + 4L * t.o00), p01 = ld4(img + 4L * t.o01);
  float4 p10 = ld4(img + 4L * t.o10), p11 = ld4(img + 4L * t.o11);
  float4 r;
  r.x = t.w00 * p00.x + t.w01 * p01.x + t.w10 * p10.x + t.w11 * p11.x;
  r.y = t.w00 * p00.y + t.w01 * p01.y + t.w10 * p10.y + t.w11 * p11.y;
  r.z = t.w00 * p00.z + t.w01 * p01.z + t.w10 * p10.z + t.w11 * p11.z;
  r.w = 0.f;
  return r;
}

// ------------------------------------------- ingest and image pyramid
// Camera blockIdx.y: the replicate-padded image (4 floats per pixel, and 8
// activations), then its quarter- and half-size copies, each sampled from
// the planar source with the same clamped coordinates: workgroups
// [0, n0) ingest, [n0, n0 + n1) quarter size, the rest half size. One launch
// for every camera's passes: at small sizes a launch costs more than its
// work (two 270x481 cameras took six launches and about 55 us with the gaps
// between them, now one and 6 us; two 720p cameras 58 -> 17 us).
struct IngestArgs {
  const float* const* src;
  int H, W, Hp, Wp;
  char* block;  // camera 0's block
  long stride;  // bytes between camera blocks
  size_t X4, Xa, L0, L1;
  int n0, n1;
};

// Pixel (y, x) of the padded image.
__device__ inline float4 padded_pixel(const float* s, int H, int W, int y, int x) {
  const long HW = (long)H * W, o = (long)min(y, H - 1) * W + min(x, W - 1);
  return make_float4(s[o], s[HW + o], s[2 * HW + o], 0.f);
}

// Bilinear sample (y, x) of the padded image resampled to Ho x Wo.
__device__ inline float4 resampled_pixel(const float* s, int H, int W, int Hp, int Wp, int Ho, int Wo, int y, int x) {
  int y0, y1, x0, x1;
  float by, ax;
  hp_tap(y, Hp, Ho, y0, y1, by);
  hp_tap(x, Wp, Wo, x0, x1, ax);
  const float4 a00 = padded_pixel(s, H, W, y0, x0), a01 = padded_pixel(s, H, W, y0, x1);
  const float4 a10 = padded_pixel(s, H, W, y1, x0), a11 = padded_pixel(s, H, W, y1, x1);
  float4 r;
  r.x = (a00.x * (1.f - ax) + a01.x * ax) * (1.f - by) + (a10.x * (1.f - ax) + a11.x * ax) * by;
  r.y = (a00.y * (1.f - ax) + a01.y * ax) * (1.f - by) + (a10.y * (1.f - ax) + a11.y * ax) * by;
  r.z = (a00.z * (1.f - ax) + a01.z * ax) * (1.f - by) + (a10.z * (1.f - ax) + a11.z * ax) * by;
  r.w = 0.f;
  return r;
}

template <typename T>
__global__ void ingest_k(IngestArgs a) {
  const int cam = blockIdx.y;
  const float* s = a.src[cam];
  char* block = a.block + cam * a.stride;
  int b = blockIdx.x;
  if (b < a.n0) {
    const long p = (long)b * TPB + threadIdx.x;
    if (p >= (long)a.Hp * a.Wp) return;
    const int y = (int)(p / a.Wp), x = (int)(p % a.Wp);
    const float4 v = padded_pixel(s, a.H, a.W, y, x);
    *reinterpret_cast<float4*>(block + a.X4 + p * 16) = v;
    const float xv[8] = {v.x, v.y, v.z, 0.f, 0.f, 0.f, 0.f, 0.f};
    store_vals<T, 8>(reinterpret_cast<T*>(block + a.Xa) + p * 8, xv);
    return;
  }
  b -= a.n0;
  const int sh = b < a.n1 ? 2 : 1;
  if (sh == 1) b -= a.n1;
  const int Ho = a.Hp >> sh, Wo = a.Wp >> sh;
  const long p = (long)b * TPB + threadIdx.x;
  if (p >= (long)Ho * Wo) return;
  const int y = (int)(p / Wo), x = (int)(p % Wo);
  *reinterpret_cast<float4*>(block + (sh == 2 ? a.L0 : a.L1) + p * 16) =
      resampled_pixel(s, a.H, a.W, a.Hp, a.Wp, Ho, Wo, y, x);
}

// ------------------------------------------------------ stage-0 input
template <typename T>
__global__ void assemble0_k(const ViewDesc* views, const CamDev* cams, int h, int w, T* x, int ld,
                            int t_plane) {
  const int v = blockIdx.y;
  const long P = (long)h * w;  // slot stride
  const long p = (long)blockIdx.x * TPB + threadIdx.x;
  const ViewDesc d = views[v];
  if (p >= (long)(d.hp >> 2) * (d.wp >> 2)) return;
  const float4 l = ld4(cams[d.cam_l].L0 + 4 * p);
  const float4 r = ld4(cams[d.cam_r].L0 + 4 * p);
  const float vals[8] = {l.x, l.y, l.z, r.x, r.y, r.z, t_plane ? d.t : 0.f, 0.f};
  store_vals<T, 8>(x + ((long)v * P + p) * ld, vals);
}

// ---------------------------------------- stage transition s -> s+1 (Eq. 2)
// FM layout: 8 floats per pixel = (F_l.x, F_l.y, F_r.x, F_r.y, M, 0, 0, 0).
template <typename T>
__global__ __launch_bounds__(TPB) void transition_k(const ViewDesc* views, const CamDev* cams, int level,
                                                    const float* FMprev, int hp, int wp, int h, int w, T* x,
                                                    int ld, float* FM, int t_plane, bool views_fast) {
  constexpr int NX = 24 * (int)sizeof(T) / 16;  // chunks of a pixel's 24 activations
  __shared__ uint4 stage[TPB * (NX + 2)];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tx, ty, v;
  super_tile(w, views_fast, tx, ty, v);
  const long P = (long)h * w;  // slot strides: P here, hp * wp for the previous level
  const ViewDesc d = views[v];
  const int vh = d.hp >> (2 - level), vw = d.wp >> (2 - level);  // this view's level sizes
  const int vhp = vh >> 1, vwp = vw >> 1;
  const int y = ty * 4 + wave, xb = tx * 64;  // the wave's first pixel
  if (y >= vh || xb >= vw) return;  // uniform over the wave; waves share nothing
  const int xx = min(xb + lane, vw - 1);  // lanes past the row's end repeat its last pixel and store nothing
  const int p = y * vw + xx;
  int y0, y1, x0, x1;
  float by, ax;
  hp_tap(y, vhp, vh, y0, y1, by);
  hp_tap(xx, vwp, vw, x0, x1, ax);
  const float* fp = FMprev + (long)v * hp * wp * 8;
  const float* q00 = fp + 8L * (y0 * vwp + x0);
  const float* q01 = fp + 8L * (y0 * vwp + x1);
  const float* q10 = fp + 8L * (y1 * vwp + x0);
  const float* q11 = fp + 8L * (y1 * vwp + x1);
  float up[5];
#pragma unroll
  for (int c = 0; c < 5; ++c)
    up[c] = (q00[c] * (1.f - ax) + q01[c] * ax) * (1.f - by) + (q10[c] * (1.f - ax) + q11[c] * ax) * by;
  const float Fx = 2.f * up[0], Fy = 2.f * up[1], Gx = 2.f * up[2], Gy = 2.f * up[3], Mt = up[4];

  const float* Lc = level == 1 ? cams[d.cam_l].L1 : cams[d.cam_l].X4;
  const float* Rc = level == 1 ? cams[d.cam_r].L1 : cams[d.cam_r].X4;
  const float4 L = ld4(Lc + 4L * p), R = ld4(Rc + 4L * p);
  const float4 Wl = sample4(Lc, warp_taps(xx, y, Fx, Fy, vw, vh));
  const float4 Wr = sample4(Rc, warp_taps(xx, y, Gx, Gy, vw, vh));

  const float vals[24] = {L.x, L.y, L.z, R.x, R.y, R.z, Wl.x, Wl.y, Wl.z, Wr.x, Wr.y, Wr.z,
                          Mt, Fx, Fy, Gx, Gy, t_plane ? d.t : 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  uint4 cx[NX];
  pack_chunks<T, 24>(vals, cx);
  const uint4 cf[2] = {make_uint4(__float_as_uint(Fx), __float_as_uint(Fy), __float_as_uint(Gx), __float_as_uint(Gy)),
                       make_uint4(__float_as_uint(Mt), 0u, 0u, 0u)};
  uint4* sx = stage + wave * 64 * NX;
  uint4* sf = stage + TPB * NX + wave * 128;
  stage_put<NX>(sx, lane, cx);
  stage_put<2>(sf, lane, cf);
  wave_sync();
  const int n_valid = min(64, vw - xb);
  const long p0 = (long)v * P + (long)y * vw + xb;
  stage_flush<NX>(sx, lane, reinterpret_cast<uint4*>(x + p0 * ld), n_valid);
  stage_flush<2>(sf, lane, reinterpret_cast<uint4*>(FM + p0 * 8), n_valid);
}

// ------------------------------------ final warp + mask blend (Eq. 1)
template <typename T>
__global__ __launch_bounds__(TPB) void final_k(const ViewDesc* views, const CamDev* cams, const float* FM,
                                               int h, int w, float* I2, T* x0u, int ld) {
  constexpr int NX = 24 * (int)sizeof(T) / 16;  // chunks of a pixel's 24 activations
  __shared__ uint4 stage[TPB * NX];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tx, ty, v;
  super_tile(w, true, tx, ty, v);
  const long P = (long)h * w;  // slot stride
  const ViewDesc d = views[v];
  const int vh = d.hp, vw = d.wp;  // this view's size
  const int y = ty * 4 + wave, xb = tx * 64;  // the wave's first pixel
  if (y >= vh || xb >= vw) return;  // uniform over the wave; waves share nothing
  // lanes past the row's end repeat its last pixel and store nothing
  const bool in = xb + lane < vw;
  const int xx = in ? xb + lane : vw - 1;
  const int p = y * vw + xx;
  const float* f = FM + ((long)v * P + p) * 8;
  const float4 F = ld4(f);
  const float M = f[4];
  const float* Lc = cams[d.cam_l].X4;
  const float* Rc = cams[d.cam_r].X4;
  const float4 L = ld4(Lc + 4L * p), R = ld4(Rc + 4L * p);
  const float4 Wl = sample4(Lc, warp_taps(xx, y, F.x, F.y, vw, vh));
  const float4 Wr = sample4(Rc, warp_taps(xx, y, F.z, F.w, vw, vh));
  const float m = 1.f / (1.f + expf(-M));
  float4 o;
  o.x = m * Wl.x + (1.f - m) * Wr.x;
  o.y = m * Wl.y + (1.f - m) * Wr.y;
  o.z = m * Wl.z + (1.f - m) * Wr.z;
  o.w = 0.f;
  if (in) store_nt(I2 + ((long)v * P + p) * 4, o);
  const float vals[24] = {L.x, L.y, L.z, R.x, R.y, R.z, Wl.x, Wl.y, Wl.z, Wr.x, Wr.y, Wr.z,
                          M, F.x, F.y, F.z, F.w, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  uint4 cx[NX];
  pack_chunks<T, 24>(vals, cx);
  uint4* sx = stage + wave * 64 * NX;
  stage_put<NX>(sx, lane, cx);
  wave_sync();
  stage_flush<NX>(sx, lane, reinterpret_cast<uint4*>(x0u + ((long)v * P + (long)y * vw + xb) * ld), min(64, vw - xb));
}

// ------------------------------- blend-only output (no refinement, Table 1)
// out = I2, cropped to H x W and written planar [3][H][W].
__global__ void blend_out_k(const float* I2, const ViewDesc* views, int Hp, int Wp, int H, int W) {
  const int v = blockIdx.y;
  const long p = (long)blockIdx.x * TPB + threadIdx.x;
  const ViewDesc d = views[v];
  if (p >= (long)d.h * d.w) return;
  const int y = (int)(p / d.w), x = (int)(p % d.w);
  const float4 b = ld4(I2 + ((long)v * Hp * Wp + (long)y * d.wp + x) * 4);
  const long HW = (long)d.h * d.w;
  float* o = d.out;
  o[p] = b.x;
  o[HW + p] = b.y;
  o[2 * HW + p] = b.z;
}

// -------------------------------------------- flow pyramid: F/2 of 2x2 mean
__device__ inline float4 flow_mean(const float4& a, const float4& c, const float4& e, const float4& g) {
  float4 r;
  r.x = 0.5f * (0.5f * (0.5f * (a.x + c.x) + 0.5f * (e.x + g.x)));
  r.y = 0.5f * (0.5f * (0.5f * (a.y + c.y) + 0.5f * (e.y + g.y)));
  r.z = 0.5f * (0.5f * (0.5f * (a.z + c.z) + 0.5f * (e.z + g.z)));
  r.w = 0.5f * (0.5f * (0.5f * (a.w + c.w) + 0.5f * (e.w + g.w)));
  return r;
}

// All four levels of a view from the full-resolution flow: a workgroup takes
// 128 x 32 full-resolution pixels (64 x 16 of level 1, in LDS, then 32 x 8,
// 16 x 4 and 8 x 2), so the coarser levels cost no launch and no second
// read (four launches of 4.6 us each at small sizes). Padded sizes are
// multiples of 16, so no 2 x 2 block crosses a border.
struct FlowArgs {
  const float* FM;  // 8 floats per pixel
  const ViewDesc* views;
  int h, w;         // slot strides: the launch's padded size
  float* F[4];
};
__global__ __launch_bounds__(TPB) void flow_pyramid_k(FlowArgs t) {
  __shared__ float4 lv[2][64 * 16];
  const int v = blockIdx.y;
  const long bx = banded_block();
  const ViewDesc d = t.views[v];
  const int tiles_x = (d.wp + 127) / 128, tiles_y = (d.hp + 31) / 32;
  if (bx >= (long)tiles_x * tiles_y) return;  // uniform over the block
  const int by = (int)(bx / tiles_x);
  const int y0 = by * 16, x0 = (int)(bx - (long)by * tiles_x) * 64;  // level-1 origin
  int vh = d.hp >> 1, vw = d.wp >> 1;
  const float* b = t.FM + (long)v * t.h * t.w * 8;
  long slot = (long)t.h * t.w >> 2;
  for (int i = threadIdx.x; i < 64 * 16; i += TPB) {
    const int y = y0 + (i >> 6), x = x0 + (i & 63);
    if (y >= vh || x >= vw) continue;
    const float* q = b + 8L * ((2 * y) * d.wp + 2 * x);
    const float4 r = flow_mean(ld4(q), ld4(q + 8), ld4(q + 8L * d.wp), ld4(q + 8L * d.wp + 8));
    lv[0][i] = r;
    *reinterpret_cast<float4*>(t.F[0] + (v * slot + (long)y * vw + x) * 4) = r;
  }
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    __syncthreads();
    vh >>= 1;
    vw >>= 1;
    slot >>= 2;
    const int tw = 64 >> k, n = (64 * 16) >> (2 * k);
    const float4* in = lv[(k - 1) & 1];
    for (int i = threadIdx.x; i < n; i += TPB) {
      const int yy = i / tw, xx = i - yy * tw;
      const int y = (y0 >> k) + yy, x = (x0 >> k) + xx;
      if (y >= vh || x >= vw) continue;
      const int o = 2 * yy * 2 * tw + 2 * xx;
      const float4 r = flow_mean(in[o], in[o + 1], in[o + 2 * tw], in[o + 2 * tw + 1]);
      lv[k & 1][i] = r;
      *reinterpret_cast<float4*>(t.F[k] + (v * slot + (long)y * vw + x) * 4) = r;
    }
  }
}

// ------------------------------------------------ context-feature warp
// One thread per (pixel, 8-channel group); groups [0, C/8) warp the left
// camera's features by F_l, groups [C/8, C/4) the right's by F_r.
// The four levels are sections of one grid (level k owns the workgroups
// first[k] .. first[k+1]-1), each in banded order over its own range.
struct CtxWarpArgs {
  const ViewDesc* views;
  const CamDev* cams;
  int h, w;  // the launch's padded full-resolution size (slot strides)
  int C[4];
  const float* flow[4];
  void* dst[4];
  int ld[4];
  long img_stride[4];
  int first[5];
};
template <typename T>
__global__ void ctx_warp_k(CtxWarpArgs t) {
  int level = 0;
#pragma unroll
  for (int k = 1; k < 4; ++k)
    if ((int)blockIdx.x >= t.first[k]) level = k;
  const int v = blockIdx.y;
  const long bx = banded(blockIdx.x - t.first[level], t.first[level + 1] - t.first[level]);
  const int C = t.C[level];
  const int G = C / 4;  // groups for both sides
  const long P = (long)(t.h >> (level + 1)) * (t.w >> (level + 1));  // slot stride
  const long id = bx * TPB + threadIdx.x;
  const ViewDesc d = t.views[v];
  const int vh = d.hp >> (level + 1), vw = d.wp >> (level + 1);  // this view's level size
  if (id >= (long)vh * vw * G) return;
  const long p = id / G;
  const int g = (int)(id - p * G);
  const bool right = g >= G / 2;
  const int c0 = (right ? g - G / 2 : g) * 8;
  const int y = (int)(p / vw), x = (int)(p % vw);
  const float4 F = ld4(t.flow[level] + ((long)v * P + p) * 4);
  const Tap4 tp = right ? warp_taps(x, y, F.z, F.w, vw, vh) : warp_taps(x, y, F.x, F.y, vw, vh);
  const T* src = reinterpret_cast<const T*>(t.cams[right ? d.cam_r : d.cam_l].ctx[level]) + c0;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  const int offs[4] = {tp.o00, tp.o01, tp.o10, tp.o11};
  const float ws[4] = {tp.w00, tp.w01, tp.w10, tp.w11};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float a[8];
    load8<T>(src + (long)offs[q] * C, a);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += ws[q] * a[i];
  }
  store_vals<T, 8>(reinterpret_cast<T*>(t.dst[level]) + (long)v * t.img_stride[level] + p * t.ld[level] +
                       (right ? C : 0) + c0,
                   acc);
}

// ----------------------------------------------------------- output head
// r = sigmoid(conv3x3(u4 -> 3)); out = clamp(I2 + 2r - 1, 0, 1), cropped and
// written planar [3][H][W]. C (the U-Net's last width) is a multiple of 8,
// at most 64, and a template parameter: each tap's C channels arrive as
// 16-byte vector loads, and the three output weights of a (tap, channel)
// are one float4 in LDS (the same address in every lane: a broadcast).
template <typename T>
__device__ inline void load_chunk(const T* p, float (&v)[16 / sizeof(T)]);

template <>
__device__ inline void load_chunk<bf16>(const bf16* p, float (&v)[8]) {
  const uint4 u = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[2 * k] = __uint_as_float(w[k] << 16);
    v[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
  }
}

template <>
__device__ inline void load_chunk<float>(const float* p, float (&v)[4]) {
  const float4 u = *reinterpret_cast<const float4*>(p);
  v[0] = u.x;
  v[1] = u.y;
  v[2] = u.z;
  v[3] = u.w;
}

template <typename T, int C>
__global__ void head_k(const T* u4, int ld, const float* wgt, const float* bias, const float* I2,
                       const ViewDesc* views, int Hp, int Wp, int H, int W) {
  constexpr int V = 16 / (int)sizeof(T);  // channels per 16-byte load
  static_assert(C % V == 0, "whole vector loads");
  __shared__ float4 ws[9 * C];  // [tap][channel] -> (w_r, w_g, w_b, 0)
  for (int i = threadIdx.x; i < 9 * C; i += TPB) {
    const int tap = i / C, c = i - tap * C;
    ws[i] = make_float4(wgt[(0 * C + c) * 9 + tap], wgt[(1 * C + c) * 9 + tap],
                        wgt[(2 * C + c) * 9 + tap], 0.f);
  }
  __syncthreads();
  const int v = blockIdx.y;
  const long bx = banded_block();
  const long p = bx * TPB + threadIdx.x;
  const ViewDesc d = views[v];
  if (p >= (long)d.h * d.w) return;
  const long slot = (long)v * Hp * Wp;  // slot stride of the launch's size
  // this view's size from here on
  H = d.h;
  W = d.w;
  Hp = d.hp;
  Wp = d.wp;
  const int y = (int)(p / W), x = (int)(p % W);
  const T* base = u4 + slot * ld;
  float z0 = bias[0], z1 = bias[1], z2 = bias[2];
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
    const int yy = y + tap / 3 - 1, xx = x + tap % 3 - 1;
    if (yy < 0 || yy >= Hp || xx < 0 || xx >= Wp) continue;  // zero padding
    const T* s = base + ((long)yy * Wp + xx) * ld;
#pragma unroll
    for (int c0 = 0; c0 < C; c0 += V) {
      float a[V];
      load_chunk<T>(s + c0, a);
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const float4 w = ws[tap * C + c0 + k];
        z0 += w.x * a[k];
        z1 += w.y * a[k];
        z2 += w.z * a[k];
      }
    }
  }
  const float4 b = ld4(I2 + (slot + (long)y * Wp + x) * 4);
  const float r0 = 1.f / (1.f + expf(-z0)), r1 = 1.f / (1.f + expf(-z1)), r2 = 1.f / (1.f + expf(-z2));
  const long HW = (long)H * W;
  float* o = d.out;
  o[p] = fminf(fmaxf(b.x + 2.f * r0 - 1.f, 0.f), 1.f);
  o[HW + p] = fminf(fmaxf(b.y + 2.f * r1 - 1.f, 0.f), 1.f);
  o[2 * HW + p] = fminf(fmaxf(b.z + 2.f * r2 - 1.f, 0.f), 1.f);
}

// The same head for bf16 activations on the matrix cores: the 3x3 conv is a
// GEMM with the 3 output channels (zero-padded to 32) as the A operand and
// 32 pixels as B, K = (tap, channel) in 16-channel MFMA steps. A wave walks
// down a strip of 32 pixels of a row, two rows a step: lane l holds the 8
// channels 8*(l/32).. of pixel l%32's three horizontal neighbours in each of
// the four rows that the two results need, of which two are loaded per step
// (one 16-byte load a tap). Each result ends with its pixels' three
// pre-activations in the first accumulators of lanes 0-31; the second row's
// move to lanes 32-63, so that all lanes share the sigmoid, the blend and the
// stores. The weights are rounded to bf16 (as every other bf16 layer's) and
// laid out once per block as MFMA fragments in LDS.
//
// Bound by the latency of its loads at four waves per SIMD (128 registers; a
// step of prefetch costs a wave and measured equal). Groups of 32 pixels that
// loaded all nine taps, divided a 64-bit index and left half the lanes idle
// in the sigmoid were bound by instructions: 4 views of 4K 832 -> 600 us (60
// bytes a pixel: 3.3 TB/s), 24 of 1080p 1196 -> 882, one of 720p 25 -> 20;
// 32 channels, 4 views of 4K 1472 -> 996.
// threads per block of the MFMA head: eight waves share one weight table
// (measured 6 % faster than four at 1080p x 112 views)
constexpr int HEAD_TPB = 512;

template <int C>
__global__ __launch_bounds__(HEAD_TPB, C == 16 ? 4 : 2) void head_mfma_k(const bf16* u4, int ld, const float* wgt,
                                                   const float* bias, const float* I2,
                                                   const ViewDesc* views, int Hp, int Wp, int rows) {
  constexpr int NC = C / 16;  // MFMAs per tap
  constexpr int WAVES = HEAD_TPB / 64;
  __shared__ uint4 wtab[9 * NC * 64];  // [tap][j][lane] weight fragments
  for (int i = threadIdx.x; i < 9 * NC * 64; i += HEAD_TPB) {
    const int ln = i & 63, tj = i >> 6, tap = tj / NC, j = tj - tap * NC;
    const int n = ln & 31, h = ln >> 5;
    bf16x8 w;
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = (bf16)(n < 3 ? wgt[(n * C + 16 * j + 8 * h + k) * 9 + tap] : 0.f);
    wtab[i] = __builtin_bit_cast(uint4, w);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lrow = lane & 31, lhalf = lane >> 5;
  const int v = blockIdx.y;
  const ViewDesc d = views[v];
  const long slot = (long)v * Hp * Wp;  // slot stride of the launch's size
  // this view's size from here on
  const int H = d.h, W = d.w, hp = d.hp, wp = d.wp;
  const int cols = (W + 31) / 32;
  const int strip = (int)banded_block() * WAVES + wave, sy = strip / cols;
  const int x0 = (strip - sy * cols) * 32, y0 = sy * rows, y1 = min(y0 + rows, H);
  if (y0 >= H) return;  // uniform over the wave
  const bf16* base = u4 + slot * ld + 8 * lhalf;
  const float bias0 = bias[0], bias1 = bias[1], bias2 = bias[2];
  const long HW = (long)H * W;
  const int x = x0 + lrow;
  // the three columns, clamped into the row, and whether they lie in it
  const bool inside = x0 > 0 && x0 + 32 < wp;  // uniform
  int xo[3];
  bool xk[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    xk[t] = x + t >= 1 && x + t <= wp;
    xo[t] = min(max(x + t - 1, 0), wp - 1) * ld;
  }
  uint4 win[4][3][NC];  // rows y - 1 .. y + 2
  auto load_row = [&](uint4 (&r)[3][NC], int yy) {
    if (yy < 0 || yy >= hp) {  // uniform: zero padding
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int j = 0; j < NC; ++j) r[t][j] = make_uint4(0u, 0u, 0u, 0u);
      return;
    }
    const bf16* src = base + (long)yy * wp * ld;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int j = 0; j < NC; ++j) r[t][j] = *reinterpret_cast<const uint4*>(src + xo[t] + 16 * j);
    if (!inside)
#pragma unroll
      for (int t = 0; t < 3; t += 2)
        if (!xk[t])
#pragma unroll
          for (int j = 0; j < NC; ++j) r[t][j] = make_uint4(0u, 0u, 0u, 0u);
  };
  load_row(win[0], y0 - 1);
  load_row(win[1], y0);
  for (int y = y0; y < y1; y += 2) {
    const int yl = y + lhalf;
    const bool in = x < W && yl < H;
    load_row(win[2], y + 1);
    load_row(win[3], y + 2);
    const float4 b = ld4(I2 + (slot + (in ? (long)yl * wp + x : 0)) * 4);
    f32x16 acc[2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[r][e] = 0.f;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const bf16x8 w = __builtin_bit_cast(bf16x8, wtab[(tap * NC + j) * 64 + lane]);
#pragma unroll
        for (int r = 0; r < 2; ++r)
          acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              w, __builtin_bit_cast(bf16x8, win[r + tap / 3][tap % 3][j]), acc[r], 0, 0, 0);
      }
    float z[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
      z[c] = __uint_as_float(
          __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[0][c]), __float_as_uint(acc[1][c]), false, false)[0]);
    z[0] += bias0;
    z[1] += bias1;
    z[2] += bias2;
    if (in) {
      const float r0 = 1.f / (1.f + expf(-z[0])), r1 = 1.f / (1.f + expf(-z[1])), r2 = 1.f / (1.f + expf(-z[2]));
      float* o = d.out + (long)yl * W + x;
      o[0] = fminf(fmaxf(b.x + 2.f * r0 - 1.f, 0.f), 1.f);
      o[HW] = fminf(fmaxf(b.y + 2.f * r1 - 1.f, 0.f), 1.f);
      o[2 * HW] = fminf(fmaxf(b.z + 2.f * r2 - 1.f, 0.f), 1.f);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int j = 0; j < NC; ++j) win[r][t][j] = win[r + 2][t][j];
  }
}

// -------------------------------------------------------- layout helpers
template <typename T>
__global__ void extract_k(const T* src, int ld, int C, long n_pix, float* dst) {
  const long p = (long)blockIdx.x * TPB + threadIdx.x;
  if (p >= n_pix) return;
  for (int c = 0; c < C; ++c) dst[c * n_pix + p] = (float)src[p * ld + c];
}

template <typename T>
__global__ void pack_nhwc_k(const float* src, int C, int H, int W, T* dst, int ld) {
  const int img = blockIdx.y;
  const long P = (long)H * W;
  const long p = (long)blockIdx.x * TPB + threadIdx.x;
  if (p >= P) return;
  const float* s = src + (long)img * C * P;
  T* o = dst + ((long)img * P + p) * ld;
  for (int c = 0; c < ld; ++c) o[c] = cvt<T>(c < C ? s[c * P + p] : 0.f);
}

inline dim3 grid1(long n, int y) { return dim3((unsigned)((n + TPB - 1) / TPB), (unsigned)y); }

}  // namespace

#define FFV_DISPATCH(dt, KERNEL, ...)                                     \
  do {                                                                     \
    if ((dt) == DType::F32)                                                \
      hipLaunchKernelGGL(KERNEL<float>, __VA_ARGS__);                      \
    else                                                                   \
      hipLaunchKernelGGL(KERNEL<bf16>, __VA_ARGS__);                       \
  } while (0)

hipError_t launch_ingest(const float* const* src, int n_cam, int H, int W, int Hp, int Wp, char* block, long stride,
                         size_t X4, size_t Xa, size_t L0, size_t L1, DType dt, hipStream_t s) {
  if (n_cam <= 0) return hipSuccess;
  const long P = (long)Hp * Wp;
  auto blocks = [](long n) { return (int)((n + TPB - 1) / TPB); };
  IngestArgs a{src, H, W, Hp, Wp, block, stride, X4, Xa, L0, L1, blocks(P), blocks(P / 16)};
  const dim3 grid((unsigned)(a.n0 + a.n1 + blocks(P / 4)), (unsigned)n_cam);
  FFV_DISPATCH(dt, ingest_k, grid, dim3(TPB), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_assemble0(const ViewDesc* views, int n_views, const CamDev* cams, int h, int w,
                            void* x, int ld, DType dt, int t_plane, hipStream_t s) {
  if (n_views <= 0) return hipSuccess;
  if (ld != 8) return hipErrorInvalidValue;  // one 16-byte-aligned run of 8 channels
  if (dt == DType::F32)
    hipLaunchKernelGGL(assemble0_k<float>, grid1((long)h * w, n_views), dim3(TPB), 0, s, views, cams,
                       h, w, (float*)x, ld, t_plane);
  else
    hipLaunchKernelGGL(assemble0_k<bf16>, grid1((long)h * w, n_views), dim3(TPB), 0, s, views, cams,
                       h, w, (bf16*)x, ld, t_plane);
  return hipGetLastError();
}

hipError_t launch_transition(const ViewDesc* views, int n_views, const CamDev* cams, int level,
                             const float* FMprev, int hp, int wp, int h, int w, void* x, int ld,
                             float* FM, DType dt, int t_plane, hipStream_t s) {
  if (n_views <= 0) return hipSuccess;
  if (ld != 24) return hipErrorInvalidValue;  // 18 channels padded to 24 (16-byte runs)
  // Views fastest up to 16 M pixels a launch; beyond, the records written are
  // gigabytes and HBM prefers fewer streams. us, views fastest / view after
  // view: 6 views of 1080p 176 / 223, 12 of 1080p (25 M pixels) 686 / 638, 4
  // of 4K 929 / 869.
  const bool fast = (long)n_views * h * w <= 16 << 20;
  if (dt == DType::F32)
    hipLaunchKernelGGL(transition_k<float>, super_grid(h, w, n_views, fast), dim3(TPB), 0, s, views, cams,
                       level, FMprev, hp, wp, h, w, (float*)x, ld, FM, t_plane, fast);
  else
    hipLaunchKernelGGL(transition_k<bf16>, super_grid(h, w, n_views, fast), dim3(TPB), 0, s, views, cams,
                       level, FMprev, hp, wp, h, w, (bf16*)x, ld, FM, t_plane, fast);
  return hipGetLastError();
}

hipError_t launch_final(const ViewDesc* views, int n_views, const CamDev* cams, const float* FM,
                        int h, int w, float* I2, void* x0u, int ld, DType dt, hipStream_t s) {
  if (n_views <= 0) return hipSuccess;
  if (ld != 24) return hipErrorInvalidValue;  // 17 channels padded to 24 (16-byte runs)
  if (dt == DType::F32)
    hipLaunchKernelGGL(final_k<float>, super_grid(h, w, n_views, true), dim3(TPB), 0, s, views, cams, FM, h,
                       w, I2, (float*)x0u, ld);
  else
    hipLaunchKernelGGL(final_k<bf16>, super_grid(h, w, n_views, true), dim3(TPB), 0, s, views, cams, FM, h,
                       w, I2, (bf16*)x0u, ld);
  return hipGetLastError();
}

hipError_t launch_flow_pyramid(const float* FM, const ViewDesc* views, int n_img, int h, int w, float* const F[4],
                               hipStream_t s) {
  if (n_img <= 0) return hipSuccess;
  if (h % 16 != 0 || w % 16 != 0) return hipErrorInvalidValue;
  const FlowArgs a{FM, views, h, w, {F[0], F[1], F[2], F[3]}};
  // (a view of a mixed batch is at most h x w, so it has no more tiles)
  const dim3 grid((unsigned)(((w + 127) / 128) * (long)((h + 31) / 32)), (unsigned)n_img);
  hipLaunchKernelGGL(flow_pyramid_k, grid, dim3(TPB), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_ctx_warp(const ViewDesc* views, int n_views, const CamDev* cams, int h, int w, const int C[4],
                           float* const flow[4], void* const dst[4], const int ld[4], DType dt, hipStream_t s) {
  if (n_views <= 0) return hipSuccess;
  CtxWarpArgs a{};
  a.views = views;
  a.cams = cams;
  a.h = h;
  a.w = w;
  for (int k = 0; k < 4; ++k) {
    const long P = (long)(h >> (k + 1)) * (w >> (k + 1));
    // 8-channel groups as 16-byte loads and stores
    if (C[k] % 8 != 0 || ld[k] % 8 != 0 || reinterpret_cast<uintptr_t>(dst[k]) % 16 != 0) return hipErrorInvalidValue;
    a.C[k] = C[k];
    a.flow[k] = flow[k];
    a.dst[k] = dst[k];
    a.ld[k] = ld[k];
    a.img_stride[k] = P * ld[k];
    const long n = (long)a.first[k] + (P * (C[k] / 4) + TPB - 1) / TPB;
    if (n > 0x7fffffffL) return hipErrorInvalidValue;
    a.first[k + 1] = (int)n;
  }
  const dim3 grid((unsigned)a.first[4], (unsigned)n_views);
  FFV_DISPATCH(dt, ctx_warp_k, grid, dim3(TPB), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_head(const void* u4, int ld, int C, const float* w, const float* b,
                       const float* I2, const ViewDesc* views, int n_img, int Hp, int Wp, int H,
                       int W, DType dt, hipStream_t s) {
  if (n_img <= 0) return hipSuccess;
  if (C <= 0 || C > 64 || C % 8 != 0 || C > ld || ld % 8 != 0) return hipErrorInvalidValue;
  if (dt == DType::BF16 && (C == 16 || C == 32)) {
    // Strips of up to 32 rows (a strip reads two more than it writes), fewer
    // where the launch would leave compute units with less than a few
    // blocks. us by rows of a strip: one view of 720p 64: 64, 32: 36, 16: 22,
    // 8 (450 blocks): 20, 4: 21; one of 1080p 32: 38, 16 (510): 33, 8: 39; 5
    // of 1136x848 32 (608): 109, 16: 93, 8: 96; 4 of 4K 32: 598, 16: 622.
    int rows = 32;
    auto blocks = [&] { return (((W + 31) / 32) * (long)((H + rows - 1) / rows) + HEAD_TPB / 64 - 1) / (HEAD_TPB / 64); };
    while (rows > 2 && blocks() * n_img < (rows > 16 ? 1024 : 384)) rows >>= 1;
    const dim3 g((unsigned)blocks(), (unsigned)n_img);
    if (C == 16)
      hipLaunchKernelGGL(head_mfma_k<16>, g, dim3(HEAD_TPB), 0, s, (const bf16*)u4, ld, w, b, I2, views, Hp, Wp, rows);
    else
      hipLaunchKernelGGL(head_mfma_k<32>, g, dim3(HEAD_TPB), 0, s, (const bf16*)u4, ld, w, b, I2, views, Hp, Wp, rows);
    return hipGetLastError();
  }
  const dim3 grid = grid1((long)H * W, n_img);
  auto go = [&](auto tc) {
    constexpr int CC = decltype(tc)::value;
    if (dt == DType::F32)
      hipLaunchKernelGGL((head_k<float, CC>), grid, dim3(TPB), 0, s, (const float*)u4, ld, w, b, I2, views,
                         Hp, Wp, H, W);
    else
      hipLaunchKernelGGL((head_k<bf16, CC>), grid, dim3(TPB), 0, s, (const bf16*)u4, ld, w, b, I2, views,
                         Hp, Wp, H, W);
  };
  switch (C) {
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 16: go(std::integral_constant<int, 16>{}); break;
    case 24: go(std::integral_constant<int, 24>{}); break;
    case 32: go(std::integral_constant<int, 32>{}); break;
    case 40: go(std::integral_constant<int, 40>{}); break;
    case 48: go(std::integral_constant<int, 48>{}); break;
    case 56: go(std::integral_constant<int, 56>{}); break;
    default: go(std::integral_constant<int, 64>{}); break;
  }
  return hipGetLastError();
}

hipError_t launch_blend_out(const float* I2, const ViewDesc* views, int n_img, int Hp, int Wp, int H,
                            int W, hipStream_t s) {
  if (n_img <= 0) return hipSuccess;
  hipLaunchKernelGGL(blend_out_k, grid1((long)H * W, n_img), dim3(TPB), 0, s, I2, views, Hp, Wp, H, W);
  return hipGetLastError();
}

hipError_t launch_extract(const void* src, DType dt, int ld, int C, long n_pix, float* dst,
                          hipStream_t s) {
  if (n_pix <= 0) return hipSuccess;
  if (dt == DType::F32)
    hipLaunchKernelGGL(extract_k<float>, grid1(n_pix, 1), dim3(TPB), 0, s, (const float*)src, ld, C,
                       n_pix, dst);
  else
    hipLaunchKernelGGL(extract_k<bf16>, grid1(n_pix, 1), dim3(TPB), 0, s, (const bf16*)src, ld, C,
                       n_pix, dst);
  return hipGetLastError();
}

hipError_t launch_pack_nhwc(const float* src, int n_img, int C, int H, int W, void* dst, int ld,
                            DType dt, hipStream_t s) {
  if (n_img <= 0) return hipSuccess;
  if (dt == DType::F32)
    hipLaunchKernelGGL(pack_nhwc_k<float>, grid1((long)H * W, n_img), dim3(TPB), 0, s, src, C, H, W,
                       (float*)dst, ld);
  else
    hipLaunchKernelGGL(pack_nhwc_k<bf16>, grid1((long)H * W, n_img), dim3(TPB), 0, s, src, C, H, W,
                       (bf16*)dst, ld);
  return hipGetLastError();
}

}  // namespace ffv
