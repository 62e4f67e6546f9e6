// Strip kernels: residual blocks that keep 65 to 96 of 128 channels inside, second convolution 3x3.
#include "strip_kernel.h"

namespace iodf {
IODF_STRIP_TABLE(kStrip433, 4, 3, 3)
}  // namespace iodf
