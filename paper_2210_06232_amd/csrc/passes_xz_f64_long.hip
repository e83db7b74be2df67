// FP64 instances of the (x, z) plane pass (k_xz) for half lengths M = 64 to 256.
#include "passes_impl.h"

namespace eifp {
EIFP_XZ_HALF(double, 64)
EIFP_XZ_HALF(double, 96)
EIFP_XZ_HALF(double, 128)
EIFP_XZ_HALF(double, 192)
EIFP_XZ_HALF(double, 256)
}
