// Strip kernels: first and last layers.
#include "strip_kernel.h"

namespace iodf {
#define IODF_STRIP_IN(NCX, NCQ, T) StripKernel{NCX, NCQ, 0, T, T, k_strip_in<NCX, NCQ, T>, nullptr}
#define IODF_STRIP_LAST(NCX, T) StripKernel{NCX, 0, 0, T, T, k_strip_last<NCX, T>, nullptr}
const StripKernel kStripIn[kStripIns] = {IODF_STRIP_IN(4, 1, 2), IODF_STRIP_IN(4, 1, 4), IODF_STRIP_IN(4, 2, 2), IODF_STRIP_IN(4, 2, 4),
                                         IODF_STRIP_IN(2, 1, 2), IODF_STRIP_IN(2, 1, 4), IODF_STRIP_IN(2, 2, 2), IODF_STRIP_IN(2, 2, 4)};
const StripKernel kStripLast[kStripLasts] = {IODF_STRIP_LAST(4, 2), IODF_STRIP_LAST(4, 4), IODF_STRIP_LAST(2, 2), IODF_STRIP_LAST(2, 4)};
}  // namespace iodf
