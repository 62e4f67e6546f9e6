// Chain kernels: residual networks whose blocks keep at most 64 of 128 channels inside, second convolution 3x3.
#include "chain_kernel.h"

namespace iodf {
IODF_CHAIN_TABLE(kChain423, 4, 2, 3)
}  // namespace iodf
