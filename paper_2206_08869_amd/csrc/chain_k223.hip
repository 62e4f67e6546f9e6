// Chain kernels: residual networks at most 64 wide, second convolution 3x3; plain networks at most 64 wide.
#include "chain_kernel.h"

namespace iodf {
IODF_CHAIN_TABLE(kChain223, 2, 2, 3)
IODF_CHAIN_TABLE(kChain20, 2, 0, 1)
}  // namespace iodf
