// Instantiations of the implicit-GEMM convolution kernel (conv_kernel.h)
// used by the library, one per N-tile class, and of the halo-reuse kernel
// (conv_halo.h). All use 128-byte K steps (conv_k_step), which the weight
// packing's K order depends on.
#include "conv_direct.h"
#include "conv_halo.h"
#include "conv_kernel.h"
#include "conv_resident.h"
#include "conv_resident_s2.h"

namespace ffv {

namespace {

// the few-channel resident kernel for the (channel chunks, N tile, stride)
// triples whose buffers fit LDS
template <typename T, int PC, int BN, int ST>
hipError_t launch_s2_pc(const ConvArgs& a, hipStream_t s) {
  if constexpr (convk::ResS2::vecs(PC, BN, ST) <= convk::ResS2::LDS_VECS)
    return convk::launch_resident_s2<T, PC, BN, ST>(a, s);
  else
    return hipErrorInvalidValue;
}

template <typename T, int BN, int ST>
hipError_t launch_s2_st(const ConvArgs& a, hipStream_t s) {
  if (a.cin_pad % 8 != 0) return hipErrorInvalidValue;
  switch (a.cin_pad / 8) {
    case 1: return launch_s2_pc<T, 1, BN, ST>(a, s);
    case 2: return launch_s2_pc<T, 2, BN, ST>(a, s);
    case 3: return launch_s2_pc<T, 3, BN, ST>(a, s);
    case 4: return launch_s2_pc<T, 4, BN, ST>(a, s);
  }
  return hipErrorInvalidValue;
}

template <typename T, int BN>
hipError_t launch_s2(const ConvArgs& a, hipStream_t s) {
  return a.stride == 1 ? launch_s2_st<T, BN, 1>(a, s) : launch_s2_st<T, BN, 2>(a, s);
}

template <typename T>
hipError_t launch_t(ConvTile tile, const ConvArgs* g, int n, hipStream_t s) {
  using namespace convk;
  // the persistent kernels take one image group
  if (!conv_tile_groupable(tile) && n != 1) return hipErrorInvalidValue;
  switch (tile) {
    case ConvTile::N256:
      return launch_variant<T, 256, 256, 4, 2, 128, 2, 1>(g, n, s);
    case ConvTile::N128:
      return launch_variant<T, 256, 128, 4, 2, 128, 2, 1>(g, n, s);
    case ConvTile::N64:
      return launch_variant<T, 256, 64, 8, 1, 128, 2, 1>(g, n, s);
    case ConvTile::N32:
      return launch_variant<T, 256, 32, 8, 1, 128, 2, 1>(g, n, s);
    case ConvTile::H32:
      return launch_halo<T>(g[0], s);
    case ConvTile::H256:
      return launch_variant<T, 256, 256, 4, 2, 128, 2, 1, true>(g, n, s);
    case ConvTile::H128:
      return launch_variant<T, 256, 128, 4, 2, 128, 2, 1, true>(g, n, s);
    case ConvTile::Q256:
      return launch_variant<T, 256, 256, 2, 4, 128, 2, 1, true>(g, n, s);
    case ConvTile::P256:
      return launch_variant<T, 256, 256, 4, 2, 128, 2, 1, true, true>(g, n, s);
    case ConvTile::R32:
      return launch_resident<T, 32>(g[0], s);
    case ConvTile::R64:
      return launch_resident<T, 64>(g[0], s);
    case ConvTile::S32:
      return launch_s2<T, 32>(g[0], s);
    case ConvTile::S64:
      return launch_s2<T, 64>(g[0], s);
    case ConvTile::S128:
      return launch_s2<T, 128>(g[0], s);
    case ConvTile::D:  // launch_conv_direct runs it
      break;
  }
  return hipErrorInvalidValue;
}

// Whether a tile's halo buffers fit LDS at a.tile_w.
template <typename T>
bool direct_fits_t(const ConvArgs& a, DirectTile tile) {
  using namespace convk;
  switch (tile) {
    case DirectTile::M64N64F:
    case DirectTile::M64N64: return direct_plan<T, 256, 64>(a, 64).nbuf > 0;
    case DirectTile::M64N128F:
    case DirectTile::M64N128: return direct_plan<T, 256, 128>(a, 64).nbuf > 0;
    case DirectTile::M128N32F:
    case DirectTile::M128N32: return direct_plan<T, 256, 32>(a, 128).nbuf > 0;
    case DirectTile::M32N32K: return direct_plan<T, 64 * kDirectParts, 32>(a, 32, true).nbuf > 0;
    case DirectTile::M128N64: return direct_plan<T, 256, 64>(a, 128).nbuf > 0;
    case DirectTile::M128N128: return direct_plan<T, 256, 128>(a, 128).nbuf > 0;
    case DirectTile::M128N256: return direct_plan<T, 512, 256>(a, 128).nbuf > 0;
    case DirectTile::M256N128: return direct_plan<T, 512, 128>(a, 256).nbuf > 0;
    default: return false;
  }
}

bool direct_fits(DType dt, const ConvArgs& a, DirectTile tile) {
  return dt == DType::F32 ? direct_fits_t<float>(a, tile)
                          : (dt == DType::BF16 ? direct_fits_t<bf16>(a, tile) : direct_fits_t<f8>(a, tile));
}

// Block width (32, 16 or 8) of the halo tiles with the least padded area for
// a launch, or 0 when the halo tiles cannot run it.
int halo_default_width(DType dt, const ConvArgs& a0) {
  int best = 0;
  long best_area = -1;
  for (int tw : {32, 16, 8}) {
    ConvArgs a = a0;
    a.tile_w = tw;
    if (!conv_halo_tile_ok(dt, a)) continue;
    const int th = 256 / tw;
    const long area = (long)((a.Ho + th - 1) / th) * th * ((a.Wo + tw - 1) / tw) * tw;
    if (best_area < 0 || area < best_area) {
      best_area = area;
      best = tw;
    }
  }
  return best;
}

}  // namespace

int conv_k_step(DType dt) { return dt == DType::F32 ? 32 : (dt == DType::BF16 ? 64 : 128); }

bool conv_halo_tile_ok(DType dt, const ConvArgs& a) { return convk::halo_tile_ok(a, conv_k_step(dt)); }

bool conv_resident_ok(DType dt, const ConvArgs& a, int bn) {
  ConvArgs b = a;
  b.tile_w = convk::Resident::TW;
  return convk::resident_ok(b, bn, (int)dtype_size(dt));
}

bool conv_resident_s2_ok(DType dt, const ConvArgs& a, int bn) {
  using convk::ResS2;
  if (a.cin_pad % 8 != 0 || a.cin_pad < 8 || a.cin_pad > 32 || (a.stride != 1 && a.stride != 2)) return false;
  const int pc = a.cin_pad / 8, st = a.stride;
  if (bn != 32 && bn != 64 && bn != 128) return false;
  return ResS2::vecs(pc, bn, st) <= ResS2::LDS_VECS && convk::resident_s2_ok(a, pc, bn, st, (int)dtype_size(dt));
}

bool conv_halo_ok(DType dt, const ConvArgs& a) {
  ConvArgs b = a;
  b.tile_w = convk::Halo::TW;
  return convk::halo_ok(b, conv_k_step(dt));
}

DirectTile conv_direct_tile(DType dt, const ConvArgs& a0, int* tile_w) {
  using namespace convk;
  const bool can = dt == DType::F32 ? direct_ok<float>(a0) : (dt == DType::BF16 ? direct_ok<bf16>(a0) : direct_ok<f8>(a0));
  if (!can) return DirectTile::None;
  struct Cand {
    DirectTile tile;
    int bm, bn;
  };
  const int rows = a0.n_rows;
  // The least padded block width of a candidate whose halo fits, and its
  // workgroups; 0 when none fits.
  auto blocks = [&](const Cand& c, int* tw_best) -> long {
    long best = 0;
    for (int tw : {16, 8, 32}) {
      ConvArgs a = a0;
      a.tile_w = tw;
      const bool fits = c.bm % tw == 0 && direct_fits(dt, a, c.tile);
      if (!fits) continue;
      const int th = c.bm / tw;
      const long n = (long)a.n_img * ((a.Ho + th - 1) / th) * ((a.Wo + tw - 1) / tw) * (a.taps == 4 ? 4 : 1) *
                     ((rows + c.bn - 1) / c.bn);
      if (best == 0 || n < best) {
        best = n;
        *tw_best = tw;
      }
    }
    return best;
  };
  const Cand m64n64{DirectTile::M64N64, 64, 64}, m64n128{DirectTile::M64N128, 64, 128},
      m128n32{DirectTile::M128N32, 128, 32}, m128n64{DirectTile::M128N64, 128, 64},
      m128n128{DirectTile::M128N128, 128, 128}, m128n256{DirectTile::M128N256, 128, 256},
      m256n128{DirectTile::M256N128, 256, 128};
  const Cand m32n32k{DirectTile::M32N32K, 32, 32}, m64n64f{DirectTile::M64N64F, 64, 64},
      m64n128f{DirectTile::M64N128F, 64, 128}, m128n32f{DirectTile::M128N32F, 128, 32};
  int tw = 0;
  long n;
  if (dt == DType::F32) {
    // Small images, several channel slices: a tile's K rounds shared by eight
    // waves (the chain of one wave's MFMAs is the launch's time). us of 32x32
    // tiles, K shared / best other tile: 256 -> 256 at 16x16 10.5 / 26, 32x32
    // (256 workgroups) 12 / 27, 32x64 (512) 23 / 30, 45x80 (920) 43 / 33;
    // stride 2, 128 -> 256, 16x16 8 / 17; transposed 256 -> 128 at 16x16 8 /
    // 15.5, 32x32 (512) 15 / 17; 128 -> 5 at 64x64 9.5 / 18. So up to 512
    // workgroups. Whether the sum is in parts goes by one image; a launch of
    // more images takes the tiles that add the same parts in turn (3 to 10 %
    // slower than those that need not). (fp32 times here and below are of
    // unscaled operands: the scaling added 2 to 6 % to every tile.)
    if (a0.cin_pad > 32 && (a0.transposed != 2 || a0.cout <= 32)) {
      n = blocks(m32n32k, &tw);
      const long n1 = a0.n_img > 0 ? n / a0.n_img : 0;
      if (n1 > 0 && n1 <= 512) {
        if (n > 512) {
          int tf = 0;
          const long nf = rows > 64 ? blocks(m64n64f, &tf) : 0;
          for (const Cand& c : {rows <= 32 ? m128n32f : rows > 64 && nf > 256 ? m64n128f : m64n64f, m64n64f})
            if (blocks(c, &tf) > 0) {
              *tile_w = tf;
              return c.tile;
            }
        }
        *tile_w = tw;
        return m32n32k.tile;
      }
    }
    // One workgroup per compute unit: the smallest tile whose workgroups fit
    // the 256 units in one round, else the largest (its weight fragments
    // feed the most MFMAs). 256 -> 256, 3x3, us of 64x64 / 64x128 / 128x128
    // tiles and of the best fp32 MFMA tile: 45x80 (228 workgroups of 64x64)
    // 33 / 42 / 68 / 80; 90x160 (226 of 128x128) 132 / 99 / 90 / 162;
    // 270x480 1098 / 915 / 823 / 1255. Narrow layers: the narrowest tile
    // (128 -> 5 transposed at 360x640: 32 columns 170, 64 columns 214).
    if (rows <= 32) {
      if (blocks(m128n32, tile_w) > 0) return m128n32.tile;
    } else if (rows <= 64) {
      n = blocks(m64n64, &tw);
      if (n > 0 && n <= 256) {
        *tile_w = tw;
        return m64n64.tile;
      }
      if (blocks(m128n64, tile_w) > 0) return m128n64.tile;
    } else {
      for (const Cand& c : {m64n64, m64n128}) {
        n = blocks(c, &tw);
        if (n > 0 && n <= 256) {
          *tile_w = tw;
          return c.tile;
        }
      }
      if (blocks(m128n128, tile_w) > 0) return m128n128.tile;
    }
    // (a halo of 2 x 64 pixels at stride 2 always fits)
    return blocks(m64n64, tile_w) > 0 ? m64n64.tile : DirectTile::None;
  }
  // bf16, fp8: launches of at most one round of workgroups, smallest tile
  // first; beyond that the tiles of ConvTile move fewer weight bytes. us of
  // 64x64 / 128x64 / 128x128 / 128x256 tiles and of the best ConvTile, 256 ->
  // 256, 3x3, bf16: 16x16 8.8 / 11 / 16 / 25 / 14; 45x80 (228 workgroups of
  // 64x64) 10.0 / 12 / 17 / 26 / 15; 68x120 (136 of 128x128) 23 / 24 / 18 /
  // 27 / 29; 135x240 (254 of 128x256) 59 / 50 / 42 / 39 / 58; 180x320 109 /
  // 97 / 79 / 71 / 66. 256x128 tiles, transposed 256 -> 128 at 90x160: 22
  // against 25. fp8 has the 64x64 tile only (the wider ones spill), worth it
  // up to two rounds: 45x80 7.9 against 10.4, 68x120 (510 workgroups) 20.5
  // against 29.3 for the default tile and 19.6 for the best.
  const Cand* list[5] = {&m64n64, nullptr, nullptr, nullptr, nullptr};
  if (dt == DType::BF16) {
    list[1] = &m128n64;
    if (rows > 64) list[2] = &m128n128;
    if (rows > 64 && a0.taps == 4) list[3] = &m256n128;
    if (rows > 128 && a0.transposed == 0 && a0.stride == 1) list[4] = &m128n256;
  }
  for (const Cand* c : list) {
    if (!c) continue;
    n = blocks(*c, &tw);
    if (n > 0 && n <= (dt == DType::FP8 ? 512 : 256)) {
      *tile_w = tw;
      return c->tile;
    }
  }
  return DirectTile::None;
}

hipError_t launch_conv_direct(DType dt, DirectTile tile, const ConvArgs& a, hipStream_t s) {
  if (a.n_img <= 0 || a.Ho <= 0 || a.Wo <= 0) return hipSuccess;
  if (dt == DType::F32) return launch_direct_f32(tile, a, s);
  return dt == DType::FP8 ? launch_direct_f8(tile, a, s) : launch_direct_bf16(tile, a, s);
}

// The figures are us per launch, one MI355X.
void conv_default_tile(DType kdt, const ConvArgs& a, ConvTile narrowest, ConvTile* tile, int* tile_w) {
  const int rows = a.n_rows;
  *tile = narrowest;  // the narrowest generic tile that holds the layer
  *tile_w = conv_tile_width(a.Ho, a.Wo);
  const bool matrix16 = kdt != DType::F32;
  const int hw = matrix16 ? halo_default_width(kdt, a) : 0;  // 0: no halo tile runs it
  auto m_tiles = [&](int tw) {
    const int th = 256 / tw;
    return (long)a.n_img * ((a.Ho + th - 1) / th) * ((a.Wo + tw - 1) / tw);
  };
  auto use = [&](ConvTile t, int tw) {
    *tile = t;
    *tile_w = tw;
  };
  // few output channels over a stride-1 3x3 neighbourhood: the persistent
  // kernel with resident weights where they fit, else the halo kernel
  if (rows <= 64 && conv_resident_ok(kdt, a, rows <= 32 ? 32 : 64)) return use(rows <= 32 ? ConvTile::R32 : ConvTile::R64, 16);
  if (rows <= 32 && conv_halo_ok(kdt, a)) return use(ConvTile::H32, 16);
  if (a.transposed == 1 && hw > 0) {
    // per-phase transposed convs: two phases (at most 128 outputs) or four
    // (at most 64) per 256-column halo tile, once those fill the chip; fp8
    // launches of at most one round of 128-column tiles take those (256 ->
    // 128 at 90x160: 16.9 against 22.4; at 180x320 57.6 against 46.6, and in
    // bf16 95 against 76, the generic tile 105)
    if (rows <= 64 && m_tiles(hw) >= 200) return use(ConvTile::Q256, hw);
    if (rows > 64 && rows <= 128)
      return use(kdt == DType::FP8 && 4 * m_tiles(hw) <= 256 ? ConvTile::H128 : ConvTile::P256, hw);
  }
  if (!a.transposed && hw > 0 && rows > 64) {
    // 3x3 stride-1 convs: with more than 128 outputs (the 256-channel
    // chains) the two-group halo tile; 128-column halo tiles for at most 128
    // outputs, and in fp8 for launches of one round of them (256 -> 256 at
    // 90x160: 22.7 against 29.9; at 135x240, 270 workgroups, 45.8 against 33.9)
    if (rows <= 128 || (kdt == DType::FP8 && m_tiles(hw) * ((rows + 127) / 128) <= 256))
      return use(ConvTile::H128, hw);
    return use(ConvTile::P256, hw);
  }
  if (!a.transposed && matrix16 && !a.out_f32 && rows <= 128 && a.cout % 8 == 0 && a.out_ld % 8 == 0) {
    // convs over a few input channels (8 to 32): the persistent kernel with
    // resident weights, narrowest N tile that holds the layer
    const int bn = rows <= 32 ? 32 : (rows <= 64 ? 64 : 128);
    if (conv_resident_s2_ok(kdt, a, bn))
      return use(bn == 32 ? ConvTile::S32 : (bn == 64 ? ConvTile::S64 : ConvTile::S128), 16);
  }
  // wide layers on small grids: narrower tiles while their workgroups fit one
  // round (fp8 128 -> 256, stride 2, 90x160 outputs: 64 columns 14.5, 128 17.4,
  // 256 23.7; 180x320: 58, 38, 28)
  if (matrix16 && rows > 64) {
    const long t = m_tiles(*tile_w) * (a.transposed == 1 ? 4 : 1);
    if (t * ((rows + 63) / 64) <= 256) return use(ConvTile::N64, *tile_w);
    if (t * ((rows + 127) / 128) <= 256) return use(ConvTile::N128, *tile_w);
  }
}

int conv_tile_width(int Ho, int Wo) {
  int best = 16;
  long best_area = -1;
  for (int tw : {16, 32, 8, 64, 128, 256}) {
    const int th = 256 / tw;
    const long area = (long)((Ho + th - 1) / th) * th * ((Wo + tw - 1) / tw) * tw;
    if (best_area < 0 || area < best_area) {
      best_area = area;
      best = tw;
    }
  }
  return best;
}

hipError_t launch_conv_grouped(DType dt, ConvTile tile, const ConvArgs* g, int n, hipStream_t s) {
  if (n < 1 || n > ConvGroup::kMax) return hipErrorInvalidValue;
  // groups with no work are left out
  ConvArgs live[ConvGroup::kMax];
  int m = 0;
  for (int i = 0; i < n; ++i)
    if (g[i].n_img > 0 && g[i].Ho > 0 && g[i].Wo > 0) live[m++] = g[i];
  if (m == 0) return hipSuccess;
  if (dt == DType::F32) return launch_t<float>(tile, live, m, s);
  if (dt == DType::FP8) return launch_t<f8>(tile, live, m, s);
  return launch_t<bf16>(tile, live, m, s);
}

hipError_t launch_conv(DType dt, ConvTile tile, const ConvArgs& a, hipStream_t s) {
  return launch_conv_grouped(dt, tile, &a, 1, s);
}

}  // namespace ffv
