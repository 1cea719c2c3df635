// The three-way bf16 split (split3.h): exact, with normal parts, over the
// whole range of weights that it takes, and the six products that the
// convolutions keep within the bound that the header states.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "split3.h"

using namespace ffv;

namespace {

int failures = 0;
void check(bool ok, const char* what, float x, float y = 0.f) {
  if (!ok && ++failures < 20) std::printf("FAILED %s: %a %a\n", what, x, y);
}

struct Parts {
  double p[3];
};

Parts split(float x) {
  uint16_t b[3];
  split3(x * kSplitScale, b);
  Parts r;
  for (int k = 0; k < 3; ++k) r.p[k] = bf2f(b[k]);
  return r;
}

void exact(float x) {
  check(splittable(x), "range", x);
  uint16_t b[3];
  split3(x * kSplitScale, b);
  double sum = 0.0;
  for (uint16_t v : b) {
    const int e = (v >> 7) & 0xff;
    check((v & 0x7fff) == 0 || (e > 0 && e < 255), "normal part", x);
    sum += bf2f(v);
  }
  check(sum == (double)x * kSplitScale, "exact", x);
  check((bf2f(b[0]) + bf2f(b[1])) + bf2f(b[2]) == x * kSplitScale, "exact in float", x);
}

double product_error(float x, float w) {
  const Parts a = split(x), b = split(w);
  const double kept = a.p[0] * b.p[0] + a.p[0] * b.p[1] + a.p[1] * b.p[0] + a.p[1] * b.p[1] + a.p[0] * b.p[2] + a.p[2] * b.p[0];
  const double want = (double)x * kSplitScale * ((double)w * kSplitScale);
  return std::fabs(kept - want) / std::fabs(want);
}

float from_bits(uint32_t u) {
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

}  // namespace

int main() {
  std::mt19937 rng(1);
  for (int i = 0; i < 4000000; ++i) {
    const float x = from_bits(rng());
    if (splittable(x)) exact(x);
  }
  // the smallest floats, subnormals, the ends of binades and of the range
  for (uint32_t u = 0; u < 70000; ++u) exact(from_bits(u));
  for (int e = -149; e <= 100; ++e)
    for (int d : {-2, -1, 0, 1, 2, 1 << 7, 1 << 14, (1 << 15) - 1, 1 << 15, (1 << 15) + 1, (1 << 16) + 1}) {
      uint32_t u;
      const float f = std::ldexp(1.f, e);
      std::memcpy(&u, &f, 4);
      const float x = from_bits(u + d);
      if (splittable(x) && u + d < 0x80000000u) {
        exact(x);
        exact(-x);
      }
    }
  check(splittable(kSplitMax), "range", kSplitMax);
  for (float x : {std::nextafter(kSplitMax, HUGE_VALF), 3.4e38f, HUGE_VALF, NAN}) {
    check(!splittable(x), "refused", x);
    check(!splittable(-x), "refused", -x);
  }

  // the six products: parts with the largest m and l, and random operands of
  // every pair of binades around 1
  double worst = 0.0;
  auto product = [&](float x, float w) {
    const double e = product_error(x, w);
    worst = e > worst ? e : worst;
    check(e <= kSplitProductError, "product", x, w);
  };
  const float corner = 1.f + 0x1p-8f - 0x1p-17f;
  product(corner, corner);
  product(-corner, 0x1p-90f * corner);
  std::uniform_real_distribution<float> u(1.f, 2.f);
  for (int i = 0; i < 4000000; ++i) product(u(rng), std::ldexp(u(rng), (int)(rng() % 40) - 20));
  std::printf("largest relative error of a product: 2^%.3f\n", std::log2(worst));
  check(worst > 0x1p-25, "the bound is near what occurs", (float)worst);
  if (failures) return 1;
  std::printf("all passed\n");
  return 0;
}
