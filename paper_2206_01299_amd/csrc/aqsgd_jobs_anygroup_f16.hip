// Shared launches of odd and wide groups instantiated for f16 activations, buffers and outputs.
#include "aqsgd_jobs_anygroup.h"

namespace aqsgd {
AQSGD_INSTANTIATE_JOBS_ANYGROUP_DTYPE(AQSGD_F16)
}
