// gemm_ring.h for (operand, output) types bf16, float.
#include "gemm_ring.h"

namespace dif {
DIF_RING_INSTANCE(bf16, float)
}  // namespace dif
