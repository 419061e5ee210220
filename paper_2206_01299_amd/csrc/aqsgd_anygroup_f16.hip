// Odd- and large-group kernels instantiated for f16 activations, buffers and outputs.
#include "aqsgd_anygroup.h"

namespace aqsgd {
AQSGD_INSTANTIATE_ANYGROUP_DTYPE(AQSGD_F16)
}
