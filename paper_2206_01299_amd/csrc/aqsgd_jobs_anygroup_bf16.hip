// Shared launches of odd and wide groups instantiated for bf16 activations, buffers and outputs.
#include "aqsgd_jobs_anygroup.h"

namespace aqsgd {
AQSGD_INSTANTIATE_JOBS_ANYGROUP_DTYPE(AQSGD_BF16)
}
