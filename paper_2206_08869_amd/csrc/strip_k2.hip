// Strip kernels: residual blocks at most 64 wide.
#include "strip_kernel.h"

namespace iodf {
IODF_STRIP_TABLE(kStrip223, 2, 2, 3)
IODF_STRIP_TABLE(kStrip221, 2, 2, 1)
}  // namespace iodf
