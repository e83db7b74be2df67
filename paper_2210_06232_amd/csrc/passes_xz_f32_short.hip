// FP32 instances of the (x, z) plane pass (k_xz) for half lengths M = 2 to 16.
#include "passes_impl.h"

namespace eifp {
EIFP_XZ_HALF(float, 2)
EIFP_XZ_HALF(float, 3)
EIFP_XZ_HALF(float, 4)
EIFP_XZ_HALF(float, 6)
EIFP_XZ_HALF(float, 8)
EIFP_XZ_HALF(float, 12)
EIFP_XZ_HALF(float, 16)
}
