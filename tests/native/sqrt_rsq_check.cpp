// Host check of the kernels' Newton step from a reciprocal root (sqrt_from_rsq in
// the library's sqrt_fix.h, included verbatim): for every float x of [1, 4), with
// y the float nearest to 1 / sqrt(x) and the floats below and above it, against
// the host's IEEE square root, and the same at both ends of the range, [2^-96,
// 2^-94) and [2^126, FLT_MAX].  Prints the pairs whose step does not round to the
// nearest, as the mantissa's float in [1, 4) and y's distance from the nearest.
//
// Built by the test with g++ -O2 -mfma -ffp-contract=off.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#define __host__
#define __device__
#include "sqrt_fix.h"

static float from_bits(uint32_t u) {
  float f;
  memcpy(&f, &u, sizeof f);
  return f;
}
static uint32_t to_bits(float f) {
  uint32_t u;
  memcpy(&u, &f, sizeof u);
  return u;
}

// The float nearest to 1 / sqrt(x), x = xi 2^-23 in [1, 4): it lies in (1/2, 1],
// a multiple of 2^-24, and 1 / sqrt(x) is below a midpoint m = k 2^-25 exactly when
// xi k^2 > 2^73.
static float nearest_rsqrt(float x) {
  if (x == 1.0f) return 1.0f;
  const uint64_t xi = (uint64_t)((double)x * 0x1p23);
  uint32_t yi = (uint32_t)(1.0 / sqrt((double)x) * 0x1p24);
  auto below = [&](uint64_t k) { return (unsigned __int128)xi * k * k > ((unsigned __int128)1 << 73); };
  while (!below(2 * (uint64_t)yi + 1)) ++yi;  // 1 / sqrt(x) above the midpoint of yi and yi + 1
  while (below(2 * (uint64_t)yi - 1)) --yi;
  return (float)yi * 0x1p-24f;
}

int main() {
  long long checked = 0, centre = 0;
  const int shifts[3] = {0, -48, 63};  // x 4^shift: [1, 4), [2^-96, 2^-94), [2^126, FLT_MAX]
  for (int s = 0; s < 3; ++s) {
    for (uint32_t u = to_bits(1.0f); u < to_bits(4.0f); ++u) {
      const float x0 = from_bits(u), y0 = nearest_rsqrt(x0);
      const float x = ldexpf(x0, 2 * shifts[s]);
      if (!(x <= 3.40282347e38f)) continue;
      const float r = sqrtf(x);
      for (int k = -1; k <= 1; ++k) {
        const float y = ldexpf(from_bits(to_bits(y0) + (uint32_t)k), -shifts[s]);
        ++checked;
        if (to_bits(sqrt_from_rsq(x, y)) == to_bits(r)) continue;
        if (k == 0) ++centre;
        printf("off range %d x 0x%08x y %+d\n", s, u, k);
      }
    }
  }
  printf("checked %lld pairs; wrong with the nearest y: %lld\n", checked, centre);
  return centre ? 1 : 0;
}
