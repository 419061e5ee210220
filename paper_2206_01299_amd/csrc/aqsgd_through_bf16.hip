// Kernels of large shared launches, which write through the L2, instantiated for bf16 activations, buffers and outputs.
#include "aqsgd_instantiate.h"

namespace aqsgd {
AQSGD_INSTANTIATE_TABLES(AQSGD_BF16, true)
}
