// Strip kernels: residual blocks that keep at most 64 of 128 channels inside, second convolution 3x3.
#include "strip_kernel.h"

namespace iodf {
IODF_STRIP_TABLE(kStrip423, 4, 2, 3)
}  // namespace iodf
