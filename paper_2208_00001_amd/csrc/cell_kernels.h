// Kernels of the thread-per-cell 3D pass (pass_cell.h), one set per tile
// geometry; each geometry is instantiated in a source file of its own.
#pragma once

#include "pass_cell.h"

namespace ggdt {

using PassKernel = void (*)(PassDesc, unsigned*, unsigned long long);

namespace dev {

// Single-channel 3D passes: one thread per box cell.
template <class Geo, bool SCANC, int RMODE, bool REC, int FMT>
__global__ __launch_bounds__(Geo::NTCAP) void pass_cell_kernel(PassDesc g, unsigned* words, unsigned long long limit) {
  __shared__ float2 pair[2 * Geo::NT];
  __shared__ int fail;
  CellLds lds{pair, nullptr, nullptr, nullptr, &fail};
  if constexpr (SCANC) {
    __shared__ float stD[Geo::STAGE];
    __shared__ float stI[Geo::STAGE];
    __shared__ float res[Geo::RES];
    lds.stD = stD;
    lds.stI = stI;
    lds.res = res;
  }
  if (ld_relaxed(words + kWordAbort) != 0u) return;
  if (g.converge && ld_relaxed(words + kWordDone) != 0u) return;  // an earlier iteration changed nothing
  run_pass_cell_mode<SCANC, RMODE, REC, Geo, FMT>(&g, g.xbuf, words, words + kWordClass, limit, lds,
                                                  xcd_remap(blockIdx.x, gridDim.x), gridDim.x);
}

template <class Geo, bool SCANC, bool REC, int FMT>
PassKernel cell_kernel_mode(int mode) {
  if (mode == kModeLam0) return pass_cell_kernel<Geo, SCANC, kModeLam0, REC, FMT>;
  if (mode == kModeLam1C1) return pass_cell_kernel<Geo, SCANC, kModeLam1C1, REC, FMT>;
  return pass_cell_kernel<Geo, SCANC, kModeGeneral, REC, FMT>;
}

// 16-bit images: plain forward passes only (no records).
template <class Geo, bool SCANC>
PassKernel cell_kernel_for(const PassDesc& d) {
  if (d.img_fmt != kImgF32) {
    if (d.rec) return nullptr;
    return d.img_fmt == kImgBF16 ? cell_kernel_mode<Geo, SCANC, false, kImgBF16>(d.mode)
                                 : cell_kernel_mode<Geo, SCANC, false, kImgF16>(d.mode);
  }
  return d.rec ? cell_kernel_mode<Geo, SCANC, true, kImgF32>(d.mode)
               : cell_kernel_mode<Geo, SCANC, false, kImgF32>(d.mode);
}

}  // namespace dev

// The kernel of a pass on its tile geometry, by source file; null if there is none.
PassKernel cell_kernel_base(const PassDesc& d);
PassKernel cell_kernel_mid(const PassDesc& d);
PassKernel cell_kernel_small(const PassDesc& d);

}  // namespace ggdt
