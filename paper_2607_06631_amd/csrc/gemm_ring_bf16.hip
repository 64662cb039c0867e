// gemm_ring.h for (operand, output) types bf16, bf16.
#include "gemm_ring.h"

namespace dif {
DIF_RING_INSTANCE(bf16, bf16)
}  // namespace dif
