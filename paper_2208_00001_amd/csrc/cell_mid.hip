// Thread-per-cell 3D pass kernels on 8 x 16 tiles.
#include "cell_kernels.h"

namespace ggdt {

PassKernel cell_kernel_mid(const PassDesc& d) {
  return dev::cell_kernel_for<dev::CellGeomMid, false>(d);
}

}  // namespace ggdt
