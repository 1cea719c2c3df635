// The exact split of a float into three bf16 parts, x = h + m + l (8 + 8 + 8
// significand bits, each the rest rounded to nearest even), with which fp32
// convolutions run on the bf16 matrix cores (the method of Henry, Tang and
// Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", ARITH 2019). Host side: the packed weights.
// Weights and activations are both scaled by 2^24 before they are split: the
// last bit of the smallest float, 2^-149, becomes 2^-125, so every non-zero
// part of every value is a normal bf16 number and the split is exact over the
// whole range (unscaled it ends at 2^-110, where l falls below the smallest
// subnormal). The sums are scaled back, which is exact too.
#pragma once

#include <cmath>
#include <cstdint>
#include <cstring>

namespace ffv {

// float -> bf16 bits, round to nearest even (NaN kept quiet).
inline uint16_t f2bf(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

inline float bf2f(uint16_t b) {
  const uint32_t u = (uint32_t)b << 16;
  float v;
  std::memcpy(&v, &u, 4);
  return v;
}

// part[0 .. 2] = h, m, l of w.
inline void split3(float w, uint16_t part[3]) {
  part[0] = f2bf(w);
  const float r = w - bf2f(part[0]);
  part[1] = f2bf(r);
  part[2] = f2bf(r - bf2f(part[1]));
}

constexpr float kSplitScale = 0x1p24f;

// Largest magnitude of a weight that is split: scaled, its parts stay well
// below the largest bf16 (h would round to infinity, m and l to minus infinity
// and NaN). Layers with larger, infinite or NaN weights run on the fp32 matrix
// instruction.
constexpr float kSplitMax = 0x1p100f;

// A product x w is summed as its six largest part products. |m| <= 2^-8 |x|
// and |l| <= 2^-17 |x|, so the dropped m l, l m and l l are at most 2^-24 +
// 2^-34 of it: one rounding of an fp32 multiplication, reached by x = w =
// 1 + 2^-8 - 2^-17. (m l and l m too would be a third more matrix work.)
constexpr double kSplitProductError = 0x1.004p-24;

inline bool splittable(float w) { return std::fabs(w) <= kSplitMax; }

}  // namespace ffv
