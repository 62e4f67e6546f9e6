// Chain kernels: residual networks at most 64 wide, second convolution 1x1.
#include "chain_kernel.h"

namespace iodf {
IODF_CHAIN_TABLE(kChain221, 2, 2, 1)
}  // namespace iodf
