// dirac_tile2d_f32.hip -- register-tile 2-D passes, FP32 state (instances of
// the kernel in dirac_tile2d_kernels.h)
#include "dirac_tile2d_kernels.h"

namespace dirac {

const void* kernel_tile2d_f32(bool strang, TileKind kind, int axes_code, int mode) {
  return kernel_tile2d<float>(strang, kind, axes_code, mode);
}

}  // namespace dirac
