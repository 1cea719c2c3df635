// Convolution kernel whose weights go straight from global memory into
// registers (gfx950), for launches the tiles of conv_kernel.h leave bound by
// latency, and for every fp32 layer.
//
// A workgroup of WM x WN waves computes BM = 32 FM WM pixels (a TH x tile_w
// block of the grid) x BN = 32 FN WN GEMM columns. The block's input halo is
// loaded into LDS a channel slice (128 bytes of every pixel) at a time with
// global_load_lds_dwordx4; as many slices as fit are resident at once
// (usually all of them), so the K loop has no barrier, or one per slice. The
// weights are packed in fragment order (fragment_order below): a wave's
// stream of 1 KiB fragments is read front to back by coalesced 16-byte loads
// D rounds ahead of their MFMAs, and no wave waits for another.
//
// K order: channel slice, tap, 16-byte chunk pairing of the two lane halves,
// as in conv_kernel.h (whose slice-major layers it shares), with one fp32
// accumulator per element for bf16 and fp8: the same results bit for bit.
//
// fp32 layers run on the bf16 matrix cores: every fp32 operand is scaled (see
// split3.h) and split exactly into three bf16 parts, x = h + m + l (8 + 8 + 8
// significand bits, each the rest rounded to nearest), activations in
// registers, weights when they are packed, and the six largest products are
// summed: h*h in one fp32 accumulator, h*m, m*h, m*m, h*l, l*h in another,
// added at the end. The three dropped ones are at most 2^-24 + 2^-34 of x*w,
// one rounding of an fp32 product (split3.h). Rounding once per 16
// products instead of once per 2, the error against float64 is smaller than
// that of v_mfma_f32_32x32x2f32: 2.2e-7 against 6.0e-7 relative (256
// channels, 3x3). A tile that meets a value the split cannot hold (infinity,
// NaN, or a magnitude past 2^104) or a sum past 2^80 gives a non-finite
// accumulator; such outputs are recomputed on the fp32 matrix instruction.
// Layers with weights that the split cannot hold (split3.h) have no weights in
// fragment order and run on the fp32 matrix instruction.
//
// What bounds it. Small grids: the chain of a workgroup's K rounds (144 for
// 256 channels): dependent MFMAs are 64 cycles apart, 3.8 us in all, and about
// 4.5 us go to the launch, the first slice and the epilogue; bf16 256 -> 256 at
// 45x80 takes 10 us where the tiles of conv_kernel.h take 15 to 65 (a barrier
// and a full load latency per K step). An fp32 round is five dependent MFMAs
// and the splitting of its activations, so small fp32 images share a tile's K
// sum among eight waves (KS): 256 -> 256 at 32x32 27 -> 12 us, at 8x8 26 -> 10.
// Larger fp32 launches: the matrix cores and power; 256 -> 256 at 270x480 took
// 823 us (1255 us on fp32 MFMA), MFMA pipes 68 % busy at 1.69 GHz, the rest
// being weight-load waits (14 %), the first slice of each workgroup and the
// epilogue. The split's VALU work runs in the shadow of the MFMAs: before it
// was interleaved by hand, the same launch took 935 us. Those fp32 figures are
// of unscaled operands; the scaling adds two multiplications to the 13
// instructions that split a pair, 1.5 % where a wave has four MFMAs per split
// (90x160 87.0 -> 88.3 us) and up to 6 % where it has one (45x80 33.2 -> 35.2).
// With it, by kernel trace on another card: 270x480 724 us = 211 TFLOP/s, on
// fp32 MFMA 1300. (Scaling once per slice in LDS cost 4 to 9 % of a view: a
// read, a multiplication and a write in a row at the slice's barrier.)
#pragma once

#include "conv_kernel.h"
#include "split3.h"

namespace ffv {
namespace convk {

// Rounds (MFMA k-groups) per tap of a slice and 16-byte weight loads per
// round and 32-column fragment.
template <typename T>
struct DirectType;
template <>
struct DirectType<bf16> {
  static constexpr int R = 4, LOADS = 1;
};
template <>
struct DirectType<f8> {
  static constexpr int R = 2, LOADS = 2;
};
template <>
struct DirectType<float> {
  static constexpr int R = 2, LOADS = 3;
};

// Input halo of a TH x TW block of outputs at stride st: hh rows of hw
// pixels. At stride 2 a row's even columns come first, so that a fragment's
// pixels read consecutive rows of the buffer at every tap.
struct DirectHalo {
  int hh, hw, ne;
  __host__ __device__ DirectHalo(int th, int tw, int st)
      : hh((th - 1) * st + 3), hw((tw - 1) * st + 3), ne(st == 2 ? tw + 1 : 0) {}
};

// Most halo loads per thread and slice of a bm-pixel block 8 to 32 wide.
constexpr int direct_loads(int bm, int st, int nt) {
  int most = 0;
  for (int tw = 8; tw <= 32; tw *= 2)
    if (bm % tw == 0) {
      const int rows = ((bm / tw - 1) * st + 3) * ((tw - 1) * st + 3), n = (rows * 8 + nt - 1) / nt;
      most = n > most ? n : most;
    }
  return most;
}

constexpr int kDirectLdsVecs = 160 * 1024 / 16;

// Parts of a K sum whose slices are shared out (KS or FOLD below), each a run
// of per slices; fewer slices than parts make one part each.
constexpr int kDirectParts = 8;

// LDS buffers of a launch: vecs 16-byte chunks each (whole loads of every
// thread), nbuf of them; 0 when not even the slices needed at once fit.
struct DirectPlan {
  int loads, vecs, nbuf, slices, per;
};
template <typename T, int NT, int BN>
inline DirectPlan direct_plan(const ConvArgs& a, int bm, bool all = false) {
  DirectPlan p{};
  const DirectHalo h(bm / a.tile_w, a.tile_w, a.stride);
  p.loads = (h.hh * h.hw * 8 + NT - 1) / NT;
  p.vecs = p.loads * NT;
  p.slices = (a.cin_pad * (int)sizeof(T) + 127) / 128;
  const int fit = (kDirectLdsVecs - 3 * BN * 4 / 16) / p.vecs;
  p.nbuf = fit < p.slices ? fit : p.slices;
  if ((p.nbuf < 2 || all) && p.nbuf < p.slices) p.nbuf = 0;
  p.per = (p.slices + kDirectParts - 1) / kDirectParts;
  return p;
}

// One third of the exact split x = h + m + l (bf16 parts, round to nearest)
// of a pair of values: stage 0 gives h and the rests, 1 m, 2 l.
__device__ inline uint32_t split_stage(float& x0, float& x1, int stage) {
  const uint32_t p = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){x0, x1}, bf16x2));
  if (stage < 2) {
    x0 -= __uint_as_float(p << 16);
    x1 -= __uint_as_float(p & 0xffff0000u);
  }
  return p;
}

// D, PA: rounds that the weights and the halo reads run ahead of the MFMAs.
// ST: stride of a 3x3 conv (1 or 2); transposed convs (4 taps per phase, or
// 9 phase-merged) use ST 1. KS: waves that share the K sum, one part each,
// added in order through LDS at the end. FOLD: the same parts one after the
// other in every wave: the same values as KS = kDirectParts.
template <typename T, int TAPS, int ST, int FM, int FN, int WM, int WN, int D, int PA, int KS = 1, bool FOLD = false>
__global__ __launch_bounds__(64 * WM * WN * KS) void conv_direct(ConvArgs a, DirectPlan pl) {
  using X = DirectType<T>;
  constexpr int NT = 64 * WM * WN * KS, BM = 32 * FM * WM, BN = 32 * FN * WN;
  static_assert(KS == 1 || (KS == kDirectParts && sizeof(T) == 4 && FM * FN * WM * WN == 1 && !FOLD), "one tile, shared K");
  static_assert(!FOLD || sizeof(T) == 4, "fp32 only");
  constexpr int R = X::R, LOADS = X::LOADS, U = TAPS * R;
  constexpr int VEC = 16 / (int)sizeof(T), BK = 128 / (int)sizeof(T);
  constexpr int LA = direct_loads(BM, ST, NT);
  constexpr bool F32 = sizeof(T) == 4;
  static_assert(U % D == 0, "the weight ring divides a slice's rounds");
  extern __shared__ __attribute__((aligned(16))) uint4 dsm[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = KS > 1 ? wave : 0;
  const int wm = KS > 1 ? 0 : wave / WN, wn = KS > 1 ? 0 : wave % WN;
  const int s0 = KS > 1 ? min(kw * pl.per, pl.slices) : 0, s1 = KS > 1 ? min(s0 + pl.per, pl.slices) : pl.slices;
  const int lrow = lane & 31, lhalf = lane >> 5;
  const bool merged = a.transposed == 2;

  // Workgroup -> (M tile, phase, N tile), N tile fastest, a contiguous range
  // per XCD: the N tiles and phases that read one halo share an L2.
  const int gx = gridDim.x, xcd = (int)blockIdx.x & 7, q8 = gx >> 3, r8 = gx & 7;
  int id = xcd * q8 + min(xcd, r8) + ((int)blockIdx.x >> 3);
  const int n_nt = (a.n_rows + BN - 1) / BN;
  const int nt = id % n_nt;
  id /= n_nt;
  int phase = 0;
  if constexpr (TAPS == 4) {
    phase = id & 3;
    id >>= 2;
  }
  const int py = phase >> 1, px = phase & 1;
  const int TW = a.tile_w, TH = BM / a.tile_w;
  const int tiles_x = (a.Wo + TW - 1) / TW, tiles_y = (a.Ho + TH - 1) / TH;
  const int img = id / (tiles_x * tiles_y);
  const int rem = id - img * tiles_x * tiles_y;
  const int ty0 = (rem / tiles_x) * TH, tx0 = (rem % tiles_x) * TW;
  const int n0 = nt * BN;

  float* prm = reinterpret_cast<float*>(dsm + pl.nbuf * pl.vecs);
  const int pbase = merged ? 0 : n0;
  float pv[3] = {0.f, 1.f, 1.f};
  static_assert(NT >= BN, "one parameter channel per thread");
  if (tid < BN && pbase + tid < a.cout) {
    pv[0] = a.bias[pbase + tid];
    if (a.w_scale) pv[1] = a.w_scale[pbase + tid];
    if (a.out_scale) pv[2] = a.out_scale[pbase + tid];
  }

  // Halo loads: load i of this thread fills chunk tid & 7 (physical) of
  // buffer row (tid + i NT) / 8; rows are XOR-swizzled by row & 7, which is
  // the same for every i (NT / 8 is a multiple of 8).
  const DirectHalo H(TH, TW, ST);
  const T* in_img = reinterpret_cast<const T*>(a.in) + (long)img * a.in_img_stride;
  const T* zero = reinterpret_cast<const T*>(a.zero);
  const int lc = (tid & 7) ^ ((tid >> 3) & 7);  // logical chunk
  int h_off[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int row = (tid + i * NT) >> 3;
    const int hy = row / H.hw, p = row - hy * H.hw;
    const int hx = ST == 2 ? (p < H.ne ? 2 * p : 2 * (p - H.ne) + 1) : p;
    const int iy = ty0 * ST - 1 + hy, ix = tx0 * ST - 1 + hx;
    const bool ok = hy < H.hh && iy >= 0 && iy < a.Hi && ix >= 0 && ix < a.Wi;
    h_off[i] = ok ? (iy * a.Wi + ix) * a.in_ld + lc * VEC : -1;
  }
  auto issue = [&](int slice, int buf) {
    const bool kin = slice * BK + lc * VEC < a.cin_pad;  // chunks past the last channel are zero
#pragma unroll
    for (int i = 0; i < LA; ++i)
      if (i < pl.loads) {
        const T* src = kin && h_off[i] >= 0 ? in_img + (h_off[i] + slice * BK) : zero;
        load_to_lds(src, dsm + buf * pl.vecs + i * NT + wave * 64);
      }
  };

  // Fragment i's pixel in the halo buffer, at tap offset 0 (stride 1: the
  // centre tap; stride 2: the first).
  int hb[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int p = (wm * FM + i) * 32 + lrow;
    const int ry = p / TW, rx = p - ry * TW;
    hb[i] = ST == 2 ? 2 * ry * H.hw + rx : (ry + 1) * H.hw + rx + 1;
  }
  auto tap_off = [&](int tap) -> int {
    if constexpr (TAPS == 4) return (py - (tap >> 1)) * H.hw + px - (tap & 1);
    const int ky = tap / 3, kx = tap % 3;
    if constexpr (ST == 2) return ky * H.hw + (kx == 1 ? H.ne : kx >> 1);
    return (ky - 1) * H.hw + kx - 1;
  };

  // Weight streams of this wave's FN column fragments: a uniform base that
  // advances and one lane offset. (The address space keeps them global
  // loads: a flat load would also hold up the LDS reads' counter.)
  typedef const __attribute__((address_space(1))) char* gptr_t;
  typedef const __attribute__((address_space(1))) __attribute__((ext_vector_type(4))) uint32_t* gvec_t;
  const int n32 = a.cout_pad / 32;
  const long stream = (long)pl.slices * U * LOADS * 1024;  // bytes per (phase, fragment)
  const uint32_t lane16 = lane * 16;
  gptr_t bp[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) bp[j] = (gptr_t)a.wfrag + ((long)phase * n32 + n0 / 32 + wn * FN + j) * stream + (long)s0 * (U * LOADS * 1024);
  auto weight = [&](int j, int k) {  // fragment k of stream j from its current place
    return __builtin_bit_cast(uint4, *(gvec_t)(bp[j] + k * 1024 + lane16));
  };

  f32x16 acc[FM][FN];
  f32x16 acc2[F32 ? FM : 1][F32 ? FN : 1];
  f32x16 tot[FOLD ? FM : 1][FOLD ? FN : 1];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[i][j][e] = 0.f;
        if constexpr (F32) acc2[i][j][e] = 0.f;
        if constexpr (FOLD) tot[i][j][e] = 0.f;
      }

  for (int s = 0; s < pl.nbuf; ++s) issue(s, s);
  uint4 fb[D][FN][LOADS];
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int l = 0; l < LOADS; ++l) fb[d][j][l] = weight(j, d * LOADS + l);
  if (tid < BN) {
    prm[tid] = pv[0];
    prm[BN + tid] = pv[1];
    prm[2 * BN + tid] = pv[2];
  }
  wait_vm<0>();
  __syncthreads();

  const char* lds = reinterpret_cast<const char*>(dsm);
  int buf = s0;
  for (int slice = s0; slice < s1; ++slice) {
    const char* ab = lds + buf * pl.vecs * 16;
    constexpr int CPR = F32 || sizeof(T) == 1 ? 2 : 1;  // A chunks per round
    int a0[FM];
    uint4 fa[PA + 1][FM][CPR];
    auto read_a = [&](int u) {
      const int r = u % R;
      if (r == 0) {
        const int off = tap_off(u / R);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const int row = hb[i] + off;
          a0[i] = (row << 7) | (((row & 7) << 4) ^ (lhalf << 6));
        }
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int c = 0; c < CPR; ++c)
          fa[u % (PA + 1)][i][c] = *reinterpret_cast<const uint4*>(ab + (a0[i] ^ ((r * CPR + c) << 4)));
    };
    // the round D ahead (the packed weights end in D rounds of padding)
    auto load_b = [&](int u, int j, int l) {
      fb[u % D][j][l] = weight(j, (u + D) * LOADS + l);
    };
#pragma unroll
    for (int u = 0; u < PA; ++u) read_a(u);
    __builtin_amdgcn_sched_barrier(0);
    // fp32: the parts of this round's and the next round's activations. The
    // next round's are split between this round's MFMAs, a third of a pair
    // (at most five VALU instructions, 20 cycles) in the shadow of each.
    uint32_t sp[2][F32 ? FM : 1][3][4];
    float x0 = 0.f, x1 = 0.f;
    auto fetch = [&](int u, int k) {  // the pair of third k
      const int i = k / 12, q = k / 3 % 4;
      const uint4& v = fa[u % (PA + 1)][i][(q >> 1) % CPR];
      x0 = __uint_as_float(q & 1 ? v.z : v.x) * kSplitScale;
      x1 = __uint_as_float(q & 1 ? v.w : v.y) * kSplitScale;
    };
    auto split = [&](int u, int k) {  // third k of round u's split
      const int i = k / 12, q = k / 3 % 4, st = k % 3;
      if (k == 0) fetch(u, 0);
      sp[u & 1][i][st][q] = split_stage(x0, x1, st);
      if (st == 2 && k + 1 < 12 * FM) fetch(u, k + 1);
    };
    if constexpr (F32)
#pragma unroll
      for (int k = 0; k < 12 * FM; ++k) split(0, k);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // The fences keep the reads PA rounds and the weight loads D rounds
      // ahead of their use (the scheduler sinks both to save registers).
      if (u + PA < U) read_a(u + PA);
      __builtin_amdgcn_sched_barrier(0);
      uint4 (&b)[FN][LOADS] = fb[u % D];
      if constexpr (F32) {
        // (weight part, activation part) of the six products; consecutive
        // MFMAs of a product have different accumulators. A weight part's
        // registers are reloaded, D rounds ahead, after its last product.
        constexpr int W[6] = {2, 0, 0, 0, 1, 1}, A[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int t = 0; t < 6 * FM * FN; ++t) {
          const int m = t / (FM * FN), i = t / FN % FM, j = t % FN, w = W[m];
          const uint32_t (&ap)[4] = sp[u & 1][i][A[m]];
          f32x16& c = m == 3 ? acc[i][j] : acc2[i][j];
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[j][w % LOADS]),
                                                      __builtin_bit_cast(bf16x8, make_uint4(ap[0], ap[1], ap[2], ap[3])),
                                                      c, 0, 0, 0);
          if (u + 1 < U)
#pragma unroll
            for (int k = 2 * t / FN; k < 2 * (t + 1) / FN; ++k) split(u + 1, k);
          if ((m == 0 || m == 3 || m == 5) && i == FM - 1) load_b(u, j, w);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            if constexpr (sizeof(T) == 1)
              mfma_f8(acc[i][j], b[j][0], b[j][1], fa[u % (PA + 1)][i][0], fa[u % (PA + 1)][i][1]);
            else
              mfma_chunk<T>(acc[i][j], b[j][0], fa[u % (PA + 1)][i][0]);
          }
      }
      if constexpr (!F32)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int l = 0; l < LOADS; ++l) load_b(u, j, l);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) bp[j] += U * LOADS * 1024;
    const int cur = buf;
    buf = buf + 1 == pl.nbuf ? 0 : buf + 1;
    if constexpr (FOLD)
      if ((slice + 1) % pl.per == 0 || slice + 1 == pl.slices)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              tot[i][j][e] += acc[i][j][e] + acc2[i][j][e];
              acc[i][j][e] = 0.f;
              acc2[i][j][e] = 0.f;
            }
    if (KS == 1 && pl.nbuf < pl.slices && slice + 1 < pl.slices) {
      // The next slice was issued at least a whole slice of weight loads
      // ago, so it has landed for this wave once those weights were used
      // (loads return in order; at most the D rounds ahead are still in
      // flight). The barrier makes every wave's share visible and frees this
      // slice's buffer.
      wait_vm<(D * FN * LOADS < 63 ? D * FN * LOADS : 63)>();
      __syncthreads();
      if (slice + pl.nbuf < pl.slices) issue(slice + pl.nbuf, cur);
    }
  }

  if constexpr (F32) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if constexpr (FOLD)
            acc[i][j][e] = tot[i][j][e];
          else
            acc[i][j][e] += acc2[i][j][e];
        }
  }
  if constexpr (KS > 1) {
    // The parts go where the halo was (a part's slice is at least twice its
    // 4 KiB); the first wave adds them and stores the tile.
    float4* part = reinterpret_cast<float4*>(dsm);
    __syncthreads();
    if (s0 < s1)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        part[(kw * 4 + g) * 64 + lane] =
            make_float4(acc[0][0][4 * g], acc[0][0][4 * g + 1], acc[0][0][4 * g + 2], acc[0][0][4 * g + 3]);
    __syncthreads();
    if (kw != 0) return;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][0][e] = 0.f;
    const int n_parts = (pl.slices + pl.per - 1) / pl.per;
    for (int k = 0; k < n_parts; ++k)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 v = part[(k * 4 + g) * 64 + lane];
        acc[0][0][4 * g] += v.x;
        acc[0][0][4 * g + 1] += v.y;
        acc[0][0][4 * g + 2] += v.z;
        acc[0][0][4 * g + 3] += v.w;
      }
  }

  // Lane l holds, for fragment (i, j), pixel i*32 + l%32 of the wave tile
  // and columns j*32 + 8g + 4*(l/32) + q (g, q = 0..3).
  const int sh = a.transposed ? 1 : 0;
  const long img_off = (long)img * a.out_img_stride;
  // (column, value) -> the output, any layout
  auto store_col = [&](long pix, int n, float v) {
    long off = pix;
    int o = n;
    if (merged) {
      const int ph = n / a.cout;
      o = n - ph * a.cout;
      off += ((long)(ph >> 1) * a.Wout + (ph & 1)) * a.out_ld;
    }
    float y = v * prm[BN + o - pbase] + prm[o - pbase];
    if (a.relu) y = fmaxf(y, 0.f);
    store_out<T>(a, off + o, o, y);
  };

  if constexpr (F32) {
    constexpr float unscale = 1.f / (kSplitScale * kSplitScale);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] *= unscale;
    auto is_bad = [&](float v) { return !(fabsf(v) <= 3.402823466e38f); };
    bool bad = false;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) bad = bad || is_bad(acc[i][j][e]);
    if (__any(bad)) {
      // The wave's tile again from unsplit operands on the fp32 matrix
      // instruction, K in the same order, read from global memory (the halo
      // ring may hold later slices only), for the outputs that are not finite;
      // the others keep their sums, so that an output does not depend on which
      // others share its wave, i.e. on the launch's tile. One loop, so that it
      // takes no registers from the ordinary path. (A view of 192 x 256 whose images
      // are infinite: 62.9 ms with one multiply-add per lane at a time, 1.85
      // so; 0.83 for ordinary images.)
      const float* x = reinterpret_cast<const float*>(in_img);
      f32x16 re[FM][FN];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) re[i][j][e] = 0.f;
      const char* ws = reinterpret_cast<const char*>(a.wfrag) + ((long)phase * n32 + n0 / 32 + wn * FN) * stream + lane16;
#pragma unroll 1
      for (int k = 0; k < pl.slices * U; ++k) {
        const int st = k / R, slice = st / TAPS, tap = st - slice * TAPS;
        const int dy = TAPS == 4 ? py - (tap >> 1) : tap / 3 - 1, dx = TAPS == 4 ? px - (tap & 1) : tap % 3 - 1;
        const int c = slice * BK + lhalf * 16 + (k - st * R) * 8;
        float4 v[FM][2];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const int p = (wm * FM + i) * 32 + lrow, ry = p / TW;
          const int iy = (ty0 + ry) * ST + dy, ix = (tx0 + p - ry * TW) * ST + dx;
          v[i][0] = v[i][1] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (iy >= 0 && iy < a.Hi && ix >= 0 && ix < a.Wi && c < a.cin_pad) {
            const float4* src = reinterpret_cast<const float4*>(x + (long)(iy * a.Wi + ix) * a.in_ld + c);
            v[i][0] = src[0];
            v[i][1] = src[1];
          }
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          uint4 part[3];
#pragma unroll
          for (int l = 0; l < 3; ++l) part[l] = *reinterpret_cast<const uint4*>(ws + j * stream + (long)(k * 3 + l) * 1024);
          float w[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float sum = 0.f;
#pragma unroll
            for (int l = 0; l < 3; ++l) {
              const uint32_t d = reinterpret_cast<const uint32_t*>(&part[l])[e >> 1];
              sum += __uint_as_float(e & 1 ? d & 0xffff0000u : d << 16);
            }
            w[e] = sum * (1.f / kSplitScale);
          }
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h)
              mfma_chunk<float>(re[i][j], make_uint4(__float_as_uint(w[4 * h]), __float_as_uint(w[4 * h + 1]),
                                                      __float_as_uint(w[4 * h + 2]), __float_as_uint(w[4 * h + 3])),
                                __builtin_bit_cast(uint4, v[i][h]));
        }
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (is_bad(acc[i][j][e])) acc[i][j][e] = re[i][j][e];
    }
  }

  // Whole runs of channels: fp32 four per store; bf16 and fp8 eight, the two
  // lane halves exchanging quads (half 0 takes the even group of a pair).
  const bool runs = !merged && !a.accumulate && a.cout % 8 == 0 && a.out_ld % 8 == 0 &&
                    ((size_t)a.out & 15) == 0 && a.out_img_stride % 8 == 0 && (F32 || !a.out_f32);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int p = (wm * FM + i) * 32 + lrow;
    const int ry = p / TW;
    const int oy = ty0 + ry, ox = tx0 + p - ry * TW;
    const bool row_ok = oy < a.Ho && ox < a.Wo;
    const long pix = img_off + ((long)((oy << sh) + py) * a.Wout + (ox << sh) + px) * a.out_ld;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int nb = n0 + (wn * FN + j) * 32 + 4 * lhalf;
      if (!runs) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int n = nb + 8 * (e >> 2) + (e & 3);
          if (row_ok && n < a.n_rows) store_col(pix, n, acc[i][j][e]);
        }
        continue;
      }
      float v[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float* pc = prm + (nb + 8 * g - n0);
        const float4 b4 = *reinterpret_cast<const float4*>(pc), s4 = *reinterpret_cast<const float4*>(pc + BN);
        const float bq[4] = {b4.x, b4.y, b4.z, b4.w}, sq[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float y = acc[i][j][4 * g + q] * sq[q] + bq[q];
          if (a.relu) y = fmaxf(y, 0.f);
          v[4 * g + q] = y;
        }
      }
      if constexpr (F32) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if (row_ok && nb + 8 * g < a.cout)
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.out) + pix + nb + 8 * g) =
                make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
      } else {
        const int c0 = n0 + (wn * FN + j) * 32 + 8 * lhalf;  // this lane's run of the first pair
        if (a.out_scale) {
          uint32_t w[4];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const float4 o4 = *reinterpret_cast<const float4*>(prm + 2 * BN + (nb + 8 * g - n0));
            w[g] = (uint32_t)to_f8(v[4 * g] * o4.x) | (uint32_t)to_f8(v[4 * g + 1] * o4.y) << 8 |
                   (uint32_t)to_f8(v[4 * g + 2] * o4.z) << 16 | (uint32_t)to_f8(v[4 * g + 3] * o4.w) << 24;
          }
#pragma unroll
          for (int g = 0; g < 4; g += 2) {
            const auto x = __builtin_amdgcn_permlane32_swap(w[g], w[g + 1], false, false);
            if (row_ok && c0 + 8 * g < a.cout)
              *reinterpret_cast<uint2*>(reinterpret_cast<uint8_t*>(a.out) + pix + c0 + 8 * g) = make_uint2(x[0], x[1]);
          }
        } else {
          uint32_t w[4][2];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            w[g][0] = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){v[4 * g], v[4 * g + 1]}, bf16x2));
            w[g][1] =
                __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){v[4 * g + 2], v[4 * g + 3]}, bf16x2));
          }
#pragma unroll
          for (int g = 0; g < 4; g += 2) {
            const auto x = __builtin_amdgcn_permlane32_swap(w[g][0], w[g + 1][0], false, false);
            const auto y = __builtin_amdgcn_permlane32_swap(w[g][1], w[g + 1][1], false, false);
            if (row_ok && c0 + 8 * g < a.cout)
              *reinterpret_cast<uint4*>(reinterpret_cast<bf16*>(a.out) + pix + c0 + 8 * g) =
                  make_uint4(x[0], y[0], x[1], y[1]);
          }
        }
      }
    }
  }
}

// Whether the kernel covers a launch (any tile width that divides the block
// is accepted; the plan decides whether the halo fits).
template <typename T>
inline bool direct_ok(const ConvArgs& a) {
  const bool nb = (a.transposed == 0 && (a.stride == 1 || a.stride == 2) && a.taps == 9) ||
                  (a.transposed == 1 && a.taps == 4 && a.stride == 1) ||
                  (a.transposed == 2 && a.taps == 9 && a.stride == 1);
  const int bk = 128 / (int)sizeof(T);
  // bf16 and fp8: slice-major layers only, the K order of the other tiles
  const bool order = sizeof(T) == 4 || a.cin_pad % bk == 0;
  return nb && order && a.wfrag && !a.amax && a.cin_pad % (16 / (int)sizeof(T)) == 0 &&
         a.in_ld % (16 / (int)sizeof(T)) == 0 && a.n_rows > 0 && a.cout_pad % 256 == 0 && a.n_rows <= a.cout_pad &&
         (a.transposed != 2 || a.n_rows == 4 * a.cout) && (long)a.Hi * a.Wi * a.in_ld < (1L << 31);
}

template <typename T, int TAPS, int ST, int FM, int FN, int WM, int WN, int D, int PA, int KS = 1, bool FOLD = false>
hipError_t launch_direct(const ConvArgs& a, hipStream_t s) {
  constexpr int NT = 64 * WM * WN * KS, BM = 32 * FM * WM, BN = 32 * FN * WN;
  if (!direct_ok<T>(a) || a.taps != TAPS || a.stride != ST || a.tile_w <= 0 || BM % a.tile_w != 0 ||
      (a.transposed == 2 && a.cout > BN))
    return hipErrorInvalidValue;
  const DirectPlan pl = direct_plan<T, NT, BN>(a, BM, KS > 1);
  if (pl.nbuf == 0 || pl.loads > direct_loads(BM, ST, NT)) return hipErrorInvalidValue;
  const int th = BM / a.tile_w;
  const long blocks = (long)a.n_img * ((a.Ho + th - 1) / th) * ((a.Wo + a.tile_w - 1) / a.tile_w) *
                      (TAPS == 4 ? 4 : 1) * ((a.n_rows + BN - 1) / BN);
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  if (blocks == 0) return hipSuccess;
  const size_t lds = (size_t)pl.nbuf * pl.vecs * 16 + 3 * BN * 4;
  hipLaunchKernelGGL((conv_direct<T, TAPS, ST, FM, FN, WM, WN, D, PA, KS, FOLD>), dim3((unsigned)blocks), dim3(NT), lds, s, a,
                     pl);
  return hipGetLastError();
}

}  // namespace convk
}  // namespace ffv
