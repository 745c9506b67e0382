// Thread-per-cell 3D pass kernels on 8 x 8 tiles.
#include "cell_kernels.h"

namespace ggdt {

PassKernel cell_kernel_small(const PassDesc& d) {
  return dev::cell_kernel_for<dev::CellGeomSmall, false>(d);
}

}  // namespace ggdt
