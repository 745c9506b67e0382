// Thread-per-cell 3D pass kernels on 16 x 16 tiles.
#include "cell_kernels.h"

namespace ggdt {

PassKernel cell_kernel_base(const PassDesc& d) {
  return d.sa == 1 ? dev::cell_kernel_for<dev::CellGeomBase, true>(d)
                   : dev::cell_kernel_for<dev::CellGeomBase, false>(d);
}

}  // namespace ggdt
