// gemm_ring.h for (operand, output) types float, float.
#include "gemm_ring.h"

namespace dif {
DIF_RING_INSTANCE(float, float)
}  // namespace dif
