// Chain kernels: residual networks whose blocks keep at most 64 of 128 channels inside, second convolution 1x1;
// plain networks 128 wide.
#include "chain_kernel.h"

namespace iodf {
IODF_CHAIN_TABLE(kChain421, 4, 2, 1)
IODF_CHAIN_TABLE(kChain40, 4, 0, 1)
}  // namespace iodf
