// Chain kernels: residual networks 128 wide inside and out, second convolution 1x1.
#include "chain_kernel.h"

namespace iodf {
IODF_CHAIN_TABLE(kChain441, 4, 4, 1)
}  // namespace iodf
