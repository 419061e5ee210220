// Kernels of single messages instantiated for f32 activations, buffers and outputs.
#include "aqsgd_single.h"

namespace aqsgd {
AQSGD_INSTANTIATE_SINGLE_DTYPE(AQSGD_F32)
}
