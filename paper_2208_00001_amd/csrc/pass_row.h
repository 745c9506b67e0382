// Lanes and edge costs of the 2D passes (pass_team.h): a row of a pass is updated
// in parallel from the previous row (FastGeodis paper, section
// "Implementation"), each lane of a wave owning one cell of the tile's row grown
// by K on both sides.  Neighbours in the previous row are the adjacent lanes,
// moved with whole-wave DPP shifts, so a step needs no barrier, no LDS and no
// index arithmetic: the serial chain of rows runs at the latency of a few VALU
// instructions per row instead of a workgroup barrier per row.
//
// Chunks of K rows use the same overlapped tiling and epoch exchange as the
// other pass kernels: the halo shrinks by one cell per row, and the tile's last
// row of a chunk is published as 64-bit exchange words (epoch << 32 | bits).
#pragma once

#include "pass_device.h"

namespace ggdt {
namespace dev {

static_assert(kRowLanes == 64 && kRowTQ == kRowLanes - 2 * kRowK, "row tile: one wave, K halo cells per side");

// Value of the lane to the left (lane - 1) / right (lane + 1), 0 past the
// wave's ends (lanes 0 and 63 are halo cells that never take part in a step).
__device__ __forceinline__ float from_left(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float from_right(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xF, 0xF, true));
}

// Edge cost through offset j from the registers of x (ix) and of its parent (iy).
template <int MODE, int NCH>
__device__ __forceinline__ float row_edge(const PassDesc& g, int j, const float* ix, const float* iy) {
  if (MODE == kModeLam0) return g.W0[j];
  const float d0 = ix[0] - iy[0];
  if (MODE == kModeLam1C1) return fabsf(d0);
  float s = d0 * d0;
#pragma unroll
  for (int c = 1; c < NCH; ++c) {
    const float dc = ix[c] - iy[c];
    s = fmaf(dc, dc, s);
  }
  return general_root<MODE, (NCH > 1)>(fmaf(g.lam, s, g.A[j]));
}

}  // namespace dev
}  // namespace ggdt
