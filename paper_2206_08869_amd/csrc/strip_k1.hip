// Strip kernels: residual blocks 128 wide, second convolution 1x1.
#include "strip_kernel.h"

namespace iodf {
IODF_STRIP_TABLE(kStrip441, 4, 4, 1)
IODF_STRIP_TABLE(kStrip421, 4, 2, 1)
}  // namespace iodf
