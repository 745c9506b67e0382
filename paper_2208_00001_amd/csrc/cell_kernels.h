// Kernels of the thread-per-cell 3D pass (pass_cell.h), one set per tile
// geometry; each geometry is instantiated in a source file of its own.
#pragma once

#include "pass_cell.h"

namespace ggdt {

using PassKernel = void (*)(PassDesc, PassSet, unsigned*, unsigned long long);

namespace dev {

// One thread per box cell.
template <class Geo, bool SCANC, int RMODE, bool REC, int FMT, int NCH>
__global__ __launch_bounds__(Geo::NTCAP) void pass_cell_kernel(PassDesc g, PassSet set, unsigned* words,
                                                               unsigned long long limit) {
  __shared__ float2 pair[2 * Geo::NT];
  __shared__ int fail;
  CellLds lds{pair, nullptr, nullptr, nullptr, nullptr, &fail};
  if constexpr (NCH > 1) {  // (lambda 0 too: it falls back to the general cost)
    __shared__ float chan[2 * (NCH - 1) * Geo::NT];
    lds.chan = chan;
  }
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
  int G;
  const int wg = pick_transform(&g, set, &G);
  run_pass_cell_mode<SCANC, RMODE, REC, Geo, FMT, NCH>(&g, g.xbuf, words, words + kWordClass, limit, lds, wg, G);
}

template <class Geo, bool SCANC, bool REC, int FMT, int NCH = 1>
PassKernel cell_kernel_mode(int mode) {
  if (mode == kModeLam0) return pass_cell_kernel<Geo, SCANC, kModeLam0, REC, FMT, NCH>;
  if (NCH == 1 && mode == kModeLam1C1) return pass_cell_kernel<Geo, SCANC, kModeLam1C1, REC, FMT, 1>;
  return pass_cell_kernel<Geo, SCANC, kModeGeneral, REC, FMT, NCH>;
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

// Multi-channel volumes, strided passes.
template <class Geo, int NCH>
PassKernel cell_kernel_channels(const PassDesc& d) {
  return d.rec ? cell_kernel_mode<Geo, false, true, kImgF32, NCH>(d.mode)
               : cell_kernel_mode<Geo, false, false, kImgF32, NCH>(d.mode);
}

}  // namespace dev

// The kernel of a pass on its tile geometry, by source file; null if there is none.
PassKernel cell_kernel_base(const PassDesc& d);
PassKernel cell_kernel_mid(const PassDesc& d);
PassKernel cell_kernel_small(const PassDesc& d);
PassKernel cell_kernel_multi(const PassDesc& d);

}  // namespace ggdt
