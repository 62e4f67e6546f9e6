// Strip kernels: first and last layers.
#include "strip_kernel.h"

namespace iodf {
const StripKernel kStripIn4[kStripEnds] = {{4, 0, 0, 2, 2, k_strip_in<4, 2>}, {4, 0, 0, 4, 4, k_strip_in<4, 4>}};
const StripKernel kStripIn2[kStripEnds] = {{2, 0, 0, 2, 2, k_strip_in<2, 2>}, {2, 0, 0, 4, 4, k_strip_in<2, 4>}};
const StripKernel kStripLast4[kStripEnds] = {{4, 0, 0, 2, 2, k_strip_last<4, 2>}, {4, 0, 0, 4, 4, k_strip_last<4, 4>}};
const StripKernel kStripLast2[kStripEnds] = {{2, 0, 0, 2, 2, k_strip_last<2, 2>}, {2, 0, 0, 4, 4, k_strip_last<2, 4>}};
}  // namespace iodf
