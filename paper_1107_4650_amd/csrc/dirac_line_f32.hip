// dirac_line_f32.hip -- register passes of FP32 lines (instances of the line
// kernel; see dirac_line_kernels.h)
#include "dirac_line_kernels.h"

namespace dirac {

const void* kernel_line_f32(bool strang, LineKind kind, int axis, int mode, int nc) {
  return kernel_line<float>(strang, kind, axis, mode, nc);
}

}  // namespace dirac
