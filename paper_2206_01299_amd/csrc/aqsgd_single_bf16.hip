// Kernels of single messages instantiated for bf16 activations, buffers and outputs.
#include "aqsgd_single.h"

namespace aqsgd {
AQSGD_INSTANTIATE_SINGLE_DTYPE(AQSGD_BF16)
}
