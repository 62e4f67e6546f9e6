// Chain kernels: residual networks whose blocks keep 65 to 96 of 128 channels inside, second convolution 3x3, on maps of
// more than 64 pixels.
#include "chain_kernel.h"

namespace iodf {
const ChainKernel kChain433[2] = {chain_kernel<4, 4, 3, 3, 4>(), chain_kernel<8, 4, 3, 3, 8>()};
}  // namespace iodf
