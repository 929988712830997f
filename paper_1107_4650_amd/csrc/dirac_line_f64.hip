// dirac_line_f64.hip -- register passes of FP64 lines (instances of the line
// kernel; see dirac_line_kernels.h)
#include "dirac_line_kernels.h"

namespace dirac {

const void* kernel_line_f64(bool strang, LineKind kind, int axis, int mode, int nc) {
  return kernel_line<double>(strang, kind, axis, mode, nc);
}

}  // namespace dirac
