// Strip kernels: residual blocks 128 wide inside and out, second convolution 3x3.
#include "strip_kernel.h"

namespace iodf {
IODF_STRIP_TABLE(kStrip443, 4, 4, 3)
}  // namespace iodf
