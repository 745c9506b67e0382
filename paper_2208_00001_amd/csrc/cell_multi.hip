// Thread-per-cell 3D pass kernels of multi-channel volumes.
#include "cell_kernels.h"

namespace ggdt {

template <class Geo>
static PassKernel channels(const PassDesc& d) {
  return d.C == 2 ? dev::cell_kernel_channels<Geo, 2>(d) : dev::cell_kernel_channels<Geo, 3>(d);
}

PassKernel cell_kernel_multi(const PassDesc& d) {
  if (d.TP == 16) return channels<dev::CellGeomBase>(d);
  return d.TQ == 16 ? channels<dev::CellGeomMid>(d) : channels<dev::CellGeomSmall>(d);
}

}  // namespace ggdt
