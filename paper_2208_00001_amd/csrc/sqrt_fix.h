// Correctly rounded square roots of floats in [2^-96, FLT_MAX].
//
// Rounding correction of a square root: given x in [2^-96, FLT_MAX] and s, a
// float within one ulp of sqrt(x), return the correctly rounded sqrtf(x); for
// x = +0 (with s = +0 or the next float) it returns +0.
//
// This is the Tuckerman rounding test, in the form Markstein gives for fused
// multiply-add hardware: with lo and hi the floats next to s, the residuals
// x - lo * s and x - hi * s, each computed with a single rounding by an fma,
// tell on which side of the midpoints (lo + s) / 2 and (s + hi) / 2 the exact
// root lies, up to a term below half an ulp that cannot change the sign.  The
// whole range has been checked exhaustively on the host for s one float below,
// at and above the correctly rounded root.
#pragma once

__host__ __device__ inline float sqrt_round_fix(float x, float s) {
  const float lo = __builtin_bit_cast(float, __builtin_bit_cast(int, s) - 1);
  const float hi = __builtin_bit_cast(float, __builtin_bit_cast(int, s) + 1);
  const float e_lo = fmaf(-lo, s, x);
  const float e_hi = fmaf(-hi, s, x);
  float r = e_lo <= 0.0f ? lo : s;
  r = e_hi > 0.0f ? hi : r;
  return r;
}

// Correctly rounded square root of x in [2^-96, FLT_MAX] from the hardware's
// reciprocal root y: g = x y is within a few ulp of the root, d = x - g^2 is
// exact up to one rounding, and g + d y / 2 rounds to the nearest (one Newton
// step; Markstein's form for fused multiply-add).  With y the float nearest to
// 1 / sqrt(x) it gives sqrtf(x) for every x of [1, 4), and by powers of 4, which
// only shift every exponent, for the whole range; with y one float off, for all
// x but those of four mantissas (five pairs of x and y), which the native test
// lists.  v_rsq_f32 is within one float of the nearest; a GPU test takes every
// float of [1, 4) through the passes, the four mantissas among them.
// In this range sqrtf as built here has the same bits (its lowering scales only
// arguments below 2^-96 and special-cases only zero and infinity).
// 5 instructions instead of sqrt_round_fix's 9: the general edge cost
// is what bounds a pass at lambda in (0, 1).
__host__ __device__ inline float sqrt_from_rsq(float x, float y) {
  const float g = x * y, h = 0.5f * y;
  return fmaf(fmaf(-g, g, x), h, g);
}
