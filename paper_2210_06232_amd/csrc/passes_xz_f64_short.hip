// FP64 instances of the (x, z) plane pass (k_xz) for half lengths M = 2 to 16.
#include "passes_impl.h"

namespace eifp {
EIFP_XZ_HALF(double, 2)
EIFP_XZ_HALF(double, 3)
EIFP_XZ_HALF(double, 4)
EIFP_XZ_HALF(double, 6)
EIFP_XZ_HALF(double, 8)
EIFP_XZ_HALF(double, 12)
EIFP_XZ_HALF(double, 16)
}
