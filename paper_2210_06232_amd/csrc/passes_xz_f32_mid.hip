// FP32 instances of the (x, z) plane pass (k_xz) for half lengths M = 24 to 48.
#include "passes_impl.h"

namespace eifp {
EIFP_XZ_HALF(float, 24)
EIFP_XZ_HALF(float, 32)
EIFP_XZ_HALF(float, 48)
}
