// dirac_tile2d_f64.hip -- register-tile 2-D passes, FP64 state (instances of
// the kernel in dirac_tile2d_kernels.h)
#include "dirac_tile2d_kernels.h"

namespace dirac {

const void* kernel_tile2d_f64(bool strang, TileKind kind, int axes_code, int mode) {
  return kernel_tile2d<double>(strang, kind, axes_code, mode);
}

}  // namespace dirac
