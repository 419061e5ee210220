// Odd- and large-group kernels instantiated for f32 activations, buffers and outputs.
#include "aqsgd_anygroup.h"

namespace aqsgd {
AQSGD_INSTANTIATE_ANYGROUP_DTYPE(AQSGD_F32)
}
