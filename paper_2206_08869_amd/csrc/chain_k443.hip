// Chain kernels: residual networks 128 wide inside and out, second convolution 3x3.
#include "chain_kernel.h"

namespace iodf {
IODF_CHAIN_TABLE(kChain443, 4, 4, 3)
}  // namespace iodf
