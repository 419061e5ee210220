// Launch table of the sparsified-backward kernels for small groups (all three dtypes).
#include "aqsgd_topk_small.h"

namespace aqsgd {

template <int DT, int MODE, int TEAM, int CPL>
static hipError_t launch_small_as(unsigned blocks, const TopkArgs& a, hipStream_t s) {
    void* data = MODE == 0 ? a.out : const_cast<void*>(a.grad);
    return launch_kernel(topk_small_kernel<DT, TEAM, CPL, MODE>, dim3(blocks), dim3(kTopkBlock), s, data, a.bitmap, a.codes,
                         a.scales, a.n_groups, a.group, a.cpg, a.keep, blocks, a.seed);
}

template <int DT, int MODE>
static hipError_t launch_small_team(TopkSmallShape shape, unsigned blocks, const TopkArgs& a, hipStream_t s) {
    switch (shape.lanes * 8 + shape.cpl) {
    case 4 * 8 + 1:  return launch_small_as<DT, MODE, 4, 1>(blocks, a, s);
    case 8 * 8 + 1:  return launch_small_as<DT, MODE, 8, 1>(blocks, a, s);
    case 8 * 8 + 2:  return launch_small_as<DT, MODE, 8, 2>(blocks, a, s);
    case 16 * 8 + 1: return launch_small_as<DT, MODE, 16, 1>(blocks, a, s);
    case 16 * 8 + 2: return launch_small_as<DT, MODE, 16, 2>(blocks, a, s);
    case 16 * 8 + 4:                                     // float32 senders and 16-bit receivers (topk_small_shape)
        if constexpr ((MODE != 0) == (DT == AQSGD_F32)) return launch_small_as<DT, MODE, 16, 4>(blocks, a, s);
        [[fallthrough]];
    default: return hipErrorInvalidValue;
    }
}

template <int DT>
static hipError_t launch_small_dt(TopkSmallShape shape, bool sender, unsigned blocks, const TopkArgs& a, hipStream_t s) {
    if (!sender) return launch_small_team<DT, 0>(shape, blocks, a, s);
    return a.stochastic ? launch_small_team<DT, 2>(shape, blocks, a, s) : launch_small_team<DT, 1>(shape, blocks, a, s);
}

hipError_t launch_topk_small(int dtype, TopkSmallShape shape, bool sender, unsigned blocks, const TopkArgs& a, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_small_dt<AQSGD_F32>(shape, sender, blocks, a, s);
    case AQSGD_F16:  return launch_small_dt<AQSGD_F16>(shape, sender, blocks, a, s);
    case AQSGD_BF16: return launch_small_dt<AQSGD_BF16>(shape, sender, blocks, a, s);
    default:         return hipErrorInvalidValue;
    }
}

}  // namespace aqsgd
