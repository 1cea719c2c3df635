// Laplacian-pyramid colour loss of the paper's training objective (section
// 3.1, "Loss functions", Eq. 3) and its gradient with respect to the
// synthesised image.
//
// Each level is linear in the image, so the pyramid is built on the
// difference D = x - gt: G^1 = D, G^(i+1) = even samples of blur(G^i), band
// L^i = G^i - expand(G^(i+1)), i = 1..5, with blur the separable binomial
// filter [1, 4, 6, 4, 1] / 16 under mirror padding (the edge sample is not
// repeated) and expand = blur with gain 2 per axis of the zero-inserted
// coarser level. The loss of an image is sum_i 2^(i-1) mean |L^i|. Every
// plane (image, channel) is an independent h x w array.
//
// Gradient: with seeds s_i = 2^(i-1) / N_i * sign(L^i) (sign 0 at 0), the
// derivative reaching G^i is a_i = s_i + R^T(a_(i+1) - E^T(s_i)), from the
// coarsest level down (a_6 = 0), where R = decimate . blur and
// E = blur_gain2 . zero-insert; the transposes gather over the taps that
// read a sample, including the mirror-folded ones.
//
// Launches. A training batch is small (8 x 256 x 448: 11 MB in, 5.5 MB out),
// so the launches count as much as the bytes. The fine levels take one
// launch each; every level of at most kTailMax samples per plane belongs to
// one workgroup per plane that keeps the rest of the pyramid in LDS (one
// launch forward, one backward). All bands run in one launch, all E^T in
// one, all partial sums in one.
// A quad (2 x 2 samples of a level, at even coordinates) belongs to one
// coarser sample, so the bands, the signs and the transposes work per quad:
// 3 x 3 coarse samples serve four fine ones, and the four signs are stored
// as one byte.
//
// Reductions: each workgroup of the band pass sums |L| of its samples in
// double (an fp32 sum of a quad already loses a row 2^-23 times as large as
// its neighbour) and writes one partial; one workgroup per image sums them in
// a fixed order in double, so the result does not depend on scheduling.
//
// Measured (one MI355X, whole call): 8 x 3 x 256 x 448 with gradient 545 ->
// 83 us, 1 x 3 x 1079 x 1917 without 2627 -> 74 us. (The bands formed in the
// tiles of the reduce passes, which saves their second read, took 90 and 75:
// the tiles' LDS work outweighs a read that hits the caches.) Before, one thread
// summed all partials of an image, each level had its own launches, seeds
// were floats, and the border gathers walked 9 x 9 taps.
#include <algorithm>

#include "common.h"
#include "lap.h"

namespace ffv {

namespace {

constexpr int TPB = 256;
// Samples per plane up to which a level is handled by the one-workgroup
// passes: 64 KB of LDS for the level and a third more for the coarser ones.
constexpr int kTailMax = 16384;
constexpr int kTailTPB = 1024;

constexpr float K0 = 1.f / 16, K1 = 4.f / 16, K2 = 6.f / 16;  // [K0 K1 K2 K1 K0]

// Levels of one call: level 0 is the image, level i + 1 halves level i.
struct Levels {
  int h[kLapLevels + 1], w[kLapLevels + 1];
};

__device__ inline int mirror(int i, int n) {
  i = i < 0 ? -i : i;
  return i > n - 1 ? 2 * (n - 1) - i : i;
}

// Weight with which output j of the mirror-padded blur along an axis of
// length n reads input i: the tap at their distance, and near an end the tap
// that the mirror folds onto i. 0 when j is no sample.
__device__ inline float blur_w(int j, int i, int n) {
  const int d = abs(i - j), lo = i + j, hi = 2 * (n - 1) - lo;
  float w = d == 0 ? K2 : (d == 1 ? K1 : (d == 2 ? K0 : 0.f));
  if (i > 0 && lo <= 2) w += lo == 2 ? K0 : K1;
  if (i < n - 1 && hi <= 2) w += hi == 2 ? K0 : K1;
  return j >= 0 && j < n ? w : 0.f;
}

// Five-tap blur of v0..v4, in tap order.
__device__ inline float blur5(float v0, float v1, float v2, float v3, float v4) {
  float r = 0.f;
  r += K0 * v0;
  r += K1 * v1;
  r += K2 * v2;
  r += K1 * v3;
  r += K0 * v4;
  return r;
}

// G^(i+1) = reduce(G^i) of one RX x RY tile of every plane; G^1 = a - b when
// DIFF. Bound by memory: the tile's input is read once into LDS (about 1.1
// reads per sample, rows of 131 consecutive floats), blurred along x there,
// then along y. (One thread per output with its 25 taps from the caches,
// two images at level 0, took 60 us for the levels of a 1079 x 1917 image.)
constexpr int RX = 64, RY = 8;
template <bool DIFF>
__global__ __launch_bounds__(TPB) void reduce_k(const float* a, const float* b, int h, int w, int ho, int wo,
                                                int tiles_x, float* out) {
  constexpr int IW = 2 * RX + 3, IH = 2 * RY + 3;
  __shared__ float in[IH][IW + 1];
  __shared__ float hr[IH][RX];
  const long plane = blockIdx.y;
  const int ty = blockIdx.x / tiles_x, tx = blockIdx.x - ty * tiles_x;
  const int x0 = tx * RX, y0 = ty * RY;
  const float* pa = a + plane * h * w;
  const float* pb = DIFF ? b + plane * h * w : nullptr;
  // (samples past the mirrored border belong to no output: clamped)
  for (int r = threadIdx.x >> 6; r < IH; r += TPB / 64) {
    const long row = (long)min(max(mirror(2 * y0 - 2 + r, h), 0), h - 1) * w;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int c = (threadIdx.x & 63) + 64 * k;
      if (c < IW) {
        const long o = row + min(max(mirror(2 * x0 - 2 + c, w), 0), w - 1);
        float v = pa[o];
        if constexpr (DIFF) v -= pb[o];
        in[r][c] = v;
      }
    }
  }
  __syncthreads();
  const int x = threadIdx.x & 63;
  for (int r = threadIdx.x >> 6; r < IH; r += TPB / 64)
    hr[r][x] = blur5(in[r][2 * x], in[r][2 * x + 1], in[r][2 * x + 2], in[r][2 * x + 3], in[r][2 * x + 4]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < RY / 4; ++k) {
    const int y = (threadIdx.x >> 6) + 4 * k;
    if (y0 + y < ho && x0 + x < wo)
      out[plane * ho * wo + (long)(y0 + y) * wo + x0 + x] =
          blur5(hr[2 * y][x], hr[2 * y + 1][x], hr[2 * y + 2][x], hr[2 * y + 3][x], hr[2 * y + 4][x]);
  }
}

// Levels m + 1 .. 5 of one plane from its level m (at most kTailMax
// samples), each level kept in LDS for the next; a chain of small steps, so
// bound by latency: one workgroup and its barriers instead of a launch per
// level.
struct TailArgs {
  Levels L;
  float* G[kLapLevels + 1];
  int m;
};
__global__ __launch_bounds__(kTailTPB) void reduce_tail_k(TailArgs t) {
  extern __shared__ float lds[];
  const long plane = blockIdx.x;
  float* cur = lds;
  const int n = t.L.h[t.m] * t.L.w[t.m];
  const float* src = t.G[t.m] + plane * n;
  for (int i = threadIdx.x; i < n; i += kTailTPB) cur[i] = src[i];
  __syncthreads();
  for (int l = t.m; l < kLapLevels; ++l) {
    const int h = t.L.h[l], w = t.L.w[l], ho = t.L.h[l + 1], wo = t.L.w[l + 1];
    float* nxt = cur + h * w;
    float* dst = t.G[l + 1] + plane * ho * wo;
    for (int i = threadIdx.x; i < ho * wo; i += kTailTPB) {
      const int y = i / wo, x = i - y * wo;
      int xs[5];
#pragma unroll
      for (int k = 0; k < 5; ++k) xs[k] = mirror(2 * x + k - 2, w);
      float r[5];
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const float* row = cur + mirror(2 * y + k - 2, h) * w;
        r[k] = blur5(row[xs[0]], row[xs[1]], row[xs[2]], row[xs[3]], row[xs[4]]);
      }
      const float v = blur5(r[0], r[1], r[2], r[3], r[4]);
      nxt[i] = v;
      dst[i] = v;
    }
    __syncthreads();
    cur = nxt;
  }
}

// The launch-wide passes over several levels: level l owns the workgroups
// first[l] .. first[l+1]-1 along grid x, one thread per quad.
struct BandArgs {
  Levels L;
  const float* x;
  const float* gt;
  const float* G[kLapLevels + 1];  // levels 1..5
  uint8_t* S[kLapLevels];          // packed signs per quad, or null
  double* partial;                 // [plane][first[5]], weighted
  double weight[kLapLevels];
  int first[kLapLevels + 1];
};
template <typename A>
__device__ inline int level_of(const A& t) {
  int l = 0;
  for (int k = 1; k < kLapLevels; ++k)
    if ((int)blockIdx.x >= t.first[k]) l = k;
  return l;
}

// Band L^i = G^i - expand(G^(i+1)) of every plane and level: per-workgroup
// partial sum of |L| and, with signs, two bits per sample (0, 1 = +, 2 = -).
// The zero-inserted samples a fine sample reads sit at even mirrored
// positions (mirroring keeps the parity), so an even row reads the coarse
// rows around it with K0, K2, K0 and an odd one the two next to it with K1.
__global__ __launch_bounds__(TPB) void band_k(BandArgs t) {
  const int l = level_of(t);
  const long plane = blockIdx.y;
  const int h = t.L.h[l], w = t.L.w[l], hn = t.L.h[l + 1], wn = t.L.w[l + 1];
  const int q = ((int)blockIdx.x - t.first[l]) * TPB + threadIdx.x;
  double sum = 0.0;
  if (q < hn * wn) {
    const int yq = q / wn, xq = q - yq * wn;
    const float* g = t.G[l + 1] + plane * hn * wn;
    const int rows[3] = {mirror(2 * yq - 2, h) >> 1, yq, mirror(2 * yq + 2, h) >> 1};
    const int cols[3] = {mirror(2 * xq - 2, w) >> 1, xq, mirror(2 * xq + 2, w) >> 1};
    float re[3], ro[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float* row = g + (long)rows[k] * wn;
      const float g0 = row[cols[0]], g1 = row[cols[1]], g2 = row[cols[2]];
      float e = 0.f, o = 0.f;
      e += K0 * g0;
      e += K2 * g1;
      e += K0 * g2;
      o += K1 * g1;
      o += K1 * g2;
      re[k] = e;
      ro[k] = o;
    }
    const float* a = l == 0 ? t.x : t.G[l];
    unsigned signs = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int y = 2 * yq + (k >> 1), x = 2 * xq + (k & 1);
      if (y >= h || x >= w) continue;
      const float* r = (k & 1) ? ro : re;
      float acc = 0.f;
      if (k >> 1) {
        acc += K1 * r[1];
        acc += K1 * r[2];
      } else {
        acc += K0 * r[0];
        acc += K2 * r[1];
        acc += K0 * r[2];
      }
      const long o = (plane * h + y) * w + x;
      float v = a[o];
      if (l == 0) v -= t.gt[o];
      const float band = v - 4.f * acc;
      sum += (double)fabsf(band);
      signs |= (band > 0.f ? 1u : (band < 0.f ? 2u : 0u)) << (2 * k);
    }
    if (t.S[l]) t.S[l][plane * hn * wn + q] = (uint8_t)signs;
  }
  // wavefront reduction, then the workgroup's four wavefronts
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  __shared__ double wsum[TPB / 64];
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < TPB / 64; ++i) s += wsum[i];
    t.partial[plane * gridDim.x + blockIdx.x] = t.weight[l] * s;
  }
}

// loss[img] = sum of the image's n partials: one workgroup per image, each
// thread a fixed strided share with its loads in flight together, then a
// fixed tree, in double. (One thread per image took 2.4 of the 2.6 ms of a
// 1079 x 1917 loss; 256 threads that walked plane by plane and level by level
// 11 us, these 4.)
constexpr int kSumTPB = 1024;
__global__ __launch_bounds__(kSumTPB) void sum_k(const double* partial, int n, float* loss) {
  const double* p = partial + (long)blockIdx.x * n;
  double total = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += kSumTPB) total += p[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
  __shared__ double red[kSumTPB / 64];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = total;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < kSumTPB / 64; ++i) s += red[i];
    loss[blockIdx.x] = (float)s;
  }
}

// E_(i+1) = E^T(s_i) on level i + 1, all levels: E^T(s)[p][q] =
// 4 * sum over fine (j, jj) of B[j][2p] B[jj][2q] s[j][jj], the 5 x 5 samples
// around (2p, 2q), i.e. 3 x 3 packed quads. Mirrored taps fold onto samples
// of that window too, so the borders differ in the weights alone.
struct EtArgs {
  Levels L;
  const uint8_t* S[kLapLevels];
  float weight[kLapLevels];
  float* E[kLapLevels + 1];  // levels 1..5
  int first[kLapLevels + 1];
  int negate_last;  // write T_5 = -E_5 in the place of E_5
};
__global__ __launch_bounds__(TPB) void et_k(EtArgs t) {
  const int l = level_of(t);
  const long plane = blockIdx.y;
  const int h = t.L.h[l], w = t.L.w[l], hn = t.L.h[l + 1], wn = t.L.w[l + 1];
  const int q = ((int)blockIdx.x - t.first[l]) * TPB + threadIdx.x;
  if (q >= hn * wn) return;
  const int y = q / wn, x = q - y * wn;
  const uint8_t* s = t.S[l] + plane * hn * wn;
  const float weight = t.weight[l];
  float wy[5] = {K0, K1, K2, K1, K0}, wx[5] = {K0, K1, K2, K1, K0};
  if (y < 2 || 2 * y + 4 > h - 1)
#pragma unroll
    for (int u = 0; u < 5; ++u) wy[u] = blur_w(2 * y - 2 + u, 2 * y, h);
  if (x < 2 || 2 * x + 4 > w - 1)
#pragma unroll
    for (int u = 0; u < 5; ++u) wx[u] = blur_w(2 * x - 2 + u, 2 * x, w);
  unsigned c[3][3];
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const uint8_t* row = s + (long)min(max(y - 1 + u, 0), hn - 1) * wn;
#pragma unroll
    for (int k = 0; k < 3; ++k) c[u][k] = row[min(max(x - 1 + k, 0), wn - 1)];
  }
  float acc = 0.f;
#pragma unroll
  for (int u = 0; u < 5; ++u) {
    float r = 0.f;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const unsigned b = (c[u >> 1][k >> 1] >> (4 * (u & 1) + 2 * (k & 1))) & 3u;
      r += wx[k] * (b == 1u ? weight : (b == 2u ? -weight : 0.f));
    }
    acc += wy[u] * r;
  }
  const float v = 4.f * acc;
  t.E[l + 1][plane * hn * wn + q] = l == kLapLevels - 1 && t.negate_last ? 0.f - v : v;
}

// The quad (yq, xq) of a_l = s_l + R^T(T_(l+1)), R^T(t)[i][ii] = sum over
// even (j, jj) of B[j][i] B[jj][ii] t[j/2][jj/2]: an even row reads the
// three coarse rows around it, an odd one the two next to it; near the
// borders only the weights differ. Level l's T_l = a_l - E_l when E is given
// (what the next finer level reads), else the gradient.
__device__ inline void rt_quad(const float* tn, const uint8_t* s, const float* E, int h, int w, int hn, int wn, int yq,
                               int xq, float weight, float* out) {
  const unsigned c = s[(long)yq * wn + xq];
  // weights of the coarse samples yq - 1, yq, yq + 1 for the even and the odd row
  float ye[3] = {K0, K2, K0}, yo[3] = {0.f, K1, K1}, xe[3] = {K0, K2, K0}, xo[3] = {0.f, K1, K1};
  if (yq < 2 || 2 * yq + 5 > h - 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      ye[k] = blur_w(2 * yq - 2 + 2 * k, 2 * yq, h);
      yo[k] = k ? blur_w(2 * yq - 2 + 2 * k, 2 * yq + 1, h) : 0.f;
    }
  if (xq < 2 || 2 * xq + 5 > w - 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      xe[k] = blur_w(2 * xq - 2 + 2 * k, 2 * xq, w);
      xo[k] = k ? blur_w(2 * xq - 2 + 2 * k, 2 * xq + 1, w) : 0.f;
    }
  const int x0 = max(xq - 1, 0), x2 = min(xq + 1, wn - 1);
  float re[3], ro[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float* row = tn + (long)min(max(yq - 1 + k, 0), hn - 1) * wn;
    float e = 0.f, o = 0.f;
    e += xe[0] * row[x0];
    e += xe[1] * row[xq];
    e += xe[2] * row[x2];
    o += xo[1] * row[xq];
    o += xo[2] * row[x2];
    re[k] = e;
    ro[k] = o;
  }
  float v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float* r = (k & 1) ? ro : re;
    float acc = 0.f;
    if (k >> 1) {
      acc += yo[1] * r[1];
      acc += yo[2] * r[2];
    } else {
      acc += ye[0] * r[0];
      acc += ye[1] * r[1];
      acc += ye[2] * r[2];
    }
    v[k] = acc;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int y = 2 * yq + (k >> 1), x = 2 * xq + (k & 1);
    if (y >= h || x >= w) continue;
    const unsigned b = (c >> (2 * k)) & 3u;
    const float a = (b == 1u ? weight : (b == 2u ? -weight : 0.f)) + v[k];
    const long o = (long)y * w + x;
    out[o] = E ? a - E[o] : a;
  }
}

__global__ __launch_bounds__(TPB) void rt_k(const float* tn, const uint8_t* s, const float* E, int h, int w, int hn,
                                            int wn, float weight, float* out) {
  const long plane = blockIdx.y;
  const int q = (int)blockIdx.x * TPB + threadIdx.x;
  if (q >= hn * wn) return;
  const int yq = q / wn;
  rt_quad(tn + plane * hn * wn, s + plane * hn * wn, E ? E + plane * h * w : nullptr, h, w, hn, wn, yq, q - yq * wn,
          weight, out + plane * h * w);
}

// T_5 .. T_m of one plane, coarsest first (T_5 = -E_5), in LDS; T_m is
// written over E_m.
struct BackTailArgs {
  Levels L;
  const uint8_t* S[kLapLevels];
  float weight[kLapLevels];
  float* E[kLapLevels + 1];
  int m;
};
__global__ __launch_bounds__(kTailTPB) void back_tail_k(BackTailArgs t) {
  extern __shared__ float lds[];
  const long plane = blockIdx.x;
  float* cur = lds;
  int n = t.L.h[kLapLevels] * t.L.w[kLapLevels];
  for (int i = threadIdx.x; i < n; i += kTailTPB) cur[i] = 0.f - t.E[kLapLevels][plane * n + i];
  __syncthreads();
  for (int l = kLapLevels - 1; l >= t.m; --l) {
    const int h = t.L.h[l], w = t.L.w[l], hn = t.L.h[l + 1], wn = t.L.w[l + 1];
    float* nxt = cur + n;
    n = h * w;
    for (int q = threadIdx.x; q < hn * wn; q += kTailTPB) {
      const int yq = q / wn;
      rt_quad(cur, t.S[l] + plane * hn * wn, t.E[l] + plane * n, h, w, hn, wn, yq, q - yq * wn, t.weight[l], nxt);
    }
    __syncthreads();
    cur = nxt;
  }
  float* dst = t.E[t.m] + plane * n;
  for (int i = threadIdx.x; i < n; i += kTailTPB) dst[i] = cur[i];
}

inline unsigned blocks(long n) { return (unsigned)((n + TPB - 1) / TPB); }

// The workspace: reduction partials, levels 1..5, and for the gradient the
// packed signs of levels 0..4 and E (later T) of levels 1..5. Each buffer
// starts on a 256-byte boundary. With base == null only the size is
// computed.
struct LapPlan {
  Levels L;
  int m;                           // finest level the one-workgroup passes own
  int first[kLapLevels + 1];       // workgroups of the all-level passes
  double* partial;
  float* G[kLapLevels + 1];
  uint8_t* S[kLapLevels];
  float* E[kLapLevels + 1];
  size_t bytes, tail_lds;
};

LapPlan lap_plan(int n_img, int H, int W, bool grad, void* base) {
  LapPlan P{};
  P.L.h[0] = H;
  P.L.w[0] = W;
  for (int i = 0; i < kLapLevels; ++i) {
    P.L.h[i + 1] = (P.L.h[i] + 1) / 2;
    P.L.w[i + 1] = (P.L.w[i] + 1) / 2;
  }
  auto samples = [&](int i) { return (long)P.L.h[i] * P.L.w[i]; };
  P.m = 1;  // (level 0 is two images, not a level buffer)
  while (P.m < kLapLevels && samples(P.m) > kTailMax) ++P.m;
  if (P.m < kLapLevels)
    for (int i = P.m; i <= kLapLevels; ++i) P.tail_lds += samples(i) * 4;
  for (int i = 0; i < kLapLevels; ++i) P.first[i + 1] = P.first[i] + (int)blocks(samples(i + 1));
  const size_t planes = 3 * (size_t)n_img;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* r = base ? static_cast<char*>(base) + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return r;
  };
  P.partial = reinterpret_cast<double*>(take(planes * P.first[kLapLevels] * 8));
  for (int i = 1; i <= kLapLevels; ++i) P.G[i] = reinterpret_cast<float*>(take(planes * samples(i) * 4));
  if (grad) {
    for (int i = 0; i < kLapLevels; ++i) P.S[i] = reinterpret_cast<uint8_t*>(take(planes * samples(i + 1)));
    for (int i = 1; i <= kLapLevels; ++i) P.E[i] = reinterpret_cast<float*>(take(planes * samples(i) * 4));
  }
  P.bytes = off;
  return P;
}

}  // namespace

size_t lap_workspace_bytes(int n_img, int H, int W, bool grad) { return lap_plan(n_img, H, W, grad, nullptr).bytes; }

hipError_t launch_lap_loss(const float* x, const float* gt, int n_img, int H, int W, float* loss, float* grad,
                           void* ws, size_t ws_bytes, hipStream_t s) {
  if (n_img <= 0) return hipSuccess;
  if (H < kLapMinSize || W < kLapMinSize || !ws) return hipErrorInvalidValue;
  const LapPlan P = lap_plan(n_img, H, W, grad != nullptr, ws);
  if (P.bytes > ws_bytes) return hipErrorInvalidValue;
  const unsigned planes = 3u * (unsigned)n_img;
  const Levels& L = P.L;
  hipError_t e;

  // forward: reduce chain, then every band and the sums (band i uses levels
  // i and i+1; level 0 is x - gt, read directly)
  for (int i = 0; i < P.m; ++i) {
    const int h = L.h[i], w = L.w[i], ho = L.h[i + 1], wo = L.w[i + 1];
    const int tx = (wo + RX - 1) / RX, ty = (ho + RY - 1) / RY;
    const dim3 grid((unsigned)(tx * ty), planes);
    if (i == 0)
      hipLaunchKernelGGL(reduce_k<true>, grid, dim3(TPB), 0, s, x, gt, h, w, ho, wo, tx, P.G[1]);
    else
      hipLaunchKernelGGL(reduce_k<false>, grid, dim3(TPB), 0, s, P.G[i], nullptr, h, w, ho, wo, tx, P.G[i + 1]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (P.m < kLapLevels) {
    TailArgs t{};
    t.L = L;
    t.m = P.m;
    for (int i = 1; i <= kLapLevels; ++i) t.G[i] = P.G[i];
    hipLaunchKernelGGL(reduce_tail_k, dim3(planes), dim3(kTailTPB), P.tail_lds, s, t);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const dim3 all((unsigned)P.first[kLapLevels], planes);
  double weight[kLapLevels];
  for (int i = 0; i < kLapLevels; ++i)
    weight[i] = (double)(1 << i) / (3.0 * (double)L.h[i] * L.w[i]);  // 2^(i-1) / N_i, N_i = 3 h w
  BandArgs b{};
  b.L = L;
  b.x = x;
  b.gt = gt;
  b.partial = P.partial;
  for (int i = 0; i <= kLapLevels; ++i) {
    b.G[i] = P.G[i];
    b.first[i] = P.first[i];
    if (i < kLapLevels) {
      b.S[i] = P.S[i];
      b.weight[i] = weight[i];
    }
  }
  hipLaunchKernelGGL(band_k, all, dim3(TPB), 0, s, b);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(sum_k, dim3((unsigned)n_img), dim3(kSumTPB), 0, s, P.partial, 3 * P.first[kLapLevels], loss);
  if ((e = hipGetLastError()) != hipSuccess || !grad) return e;

  // backward: E^T of every level's signs, then T coarsest level first
  EtArgs t{};
  BackTailArgs k{};
  t.L = k.L = L;
  k.m = P.m;
  for (int i = 0; i <= kLapLevels; ++i) {
    t.E[i] = k.E[i] = P.E[i];
    t.first[i] = P.first[i];
    if (i < kLapLevels) {
      t.S[i] = k.S[i] = P.S[i];
      t.weight[i] = k.weight[i] = (float)weight[i];
    }
  }
  // (images whose level 5 is larger than the one-workgroup pass takes have
  // no such pass)
  t.negate_last = P.m == kLapLevels;
  hipLaunchKernelGGL(et_k, all, dim3(TPB), 0, s, t);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (P.m < kLapLevels) {
    hipLaunchKernelGGL(back_tail_k, dim3(planes), dim3(kTailTPB), P.tail_lds, s, k);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  for (int i = P.m - 1; i >= 0; --i) {
    // T_i replaces E_i, sample by sample; level 0 gives the gradient
    hipLaunchKernelGGL(rt_k, dim3(blocks((long)L.h[i + 1] * L.w[i + 1]), planes), dim3(TPB), 0, s, P.E[i + 1], P.S[i],
                       P.E[i], L.h[i], L.w[i], L.h[i + 1], L.w[i + 1], (float)weight[i], i == 0 ? grad : P.E[i]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ffv
