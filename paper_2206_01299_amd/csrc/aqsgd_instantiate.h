// Launch tables of one storage dtype: every (rounding, team shape, kind) of the job
// kernel that hosts quantising jobs and every unroll of the one that holds
// dequantising jobs alone.  Each dtype gets its own translation unit so the three
// compile in parallel.
#pragma once

#include "aqsgd_kernels.h"

namespace aqsgd {

template <int DT, int ROUND, int KIND, int TEAM, int CPL>
static hipError_t launch_cj(const JobTable& t, hipStream_t stream) {
    constexpr int threads = TEAM > kWave ? TEAM : kBlock;
    // Teams of a wavefront and more loop only where a cap on the grid asks for it: one kernel does.
    if constexpr (KIND == kTableLoops && TEAM >= kWave) return launch_cj<DT, ROUND, kTableLoopsThree, TEAM, CPL>(t, stream);
    else return launch_kernel(codec_jobs_kernel<DT, ROUND, TEAM, CPL, KIND>, dim3(t.total_blocks), dim3(threads),
                              stream, t);
}

template <int DT, int ROUND, int KIND>
static hipError_t launch_cj_shape(int shape, const JobTable& t, hipStream_t stream) {
    switch (shape) {
    case kTeam8x1:    return launch_cj<DT, ROUND, KIND, 8, 1>(t, stream);
    case kTeam16x1:   return launch_cj<DT, ROUND, KIND, 16, 1>(t, stream);
    case kTeam32x1:   return launch_cj<DT, ROUND, KIND, 32, 1>(t, stream);
    case kTeam64x1:   return launch_cj<DT, ROUND, KIND, 64, 1>(t, stream);
    case kTeam64x2:   return launch_cj<DT, ROUND, KIND, 64, 2>(t, stream);
    case kTeam64x3:   return launch_cj<DT, ROUND, KIND, 64, 3>(t, stream);
    case kTeam64x4:   return launch_cj<DT, ROUND, KIND, 64, 4>(t, stream);
    case kTeam256x2:  return launch_cj<DT, ROUND, KIND, 256, 2>(t, stream);
    case kTeam256x4:  return launch_cj<DT, ROUND, KIND, 256, 4>(t, stream);
    case kTeam1024x2: return launch_cj<DT, ROUND, KIND, 1024, 2>(t, stream);
    case kTeam1024x4: return launch_cj<DT, ROUND, KIND, 1024, 4>(t, stream);
    default:          return hipErrorInvalidValue;
    }
}

template <int DT, int ROUND>
static hipError_t launch_cj_kind(int shape, TableKind kind, const JobTable& t, hipStream_t stream) {
    switch (kind) {
    case kTableOneStep:      return launch_cj_shape<DT, ROUND, kTableOneStep>(shape, t, stream);
    case kTableOneStepThree: return launch_cj_shape<DT, ROUND, kTableOneStepThree>(shape, t, stream);
    case kTableLoops:        return launch_cj_shape<DT, ROUND, kTableLoops>(shape, t, stream);
    case kTableLoopsThree:   return launch_cj_shape<DT, ROUND, kTableLoopsThree>(shape, t, stream);
    default:                 return hipErrorInvalidValue;
    }
}

template <int DT>
hipError_t launch_codec_jobs_dt(int rounding, int shape, TableKind kind, const JobTable& t, hipStream_t stream) {
    return rounding == AQSGD_ROUND_STOCHASTIC
               ? launch_cj_kind<DT, AQSGD_ROUND_STOCHASTIC>(shape, kind, t, stream)
               : launch_cj_kind<DT, AQSGD_ROUND_NEAREST>(shape, kind, t, stream);
}

template <int DT>
hipError_t launch_dequant_jobs_dt(int unroll, const JobTable& t, hipStream_t stream) {
    const dim3 grid(t.total_blocks), block(kBlock);
    switch (unroll) {
    case 1: return launch_kernel(dequant_jobs_kernel<DT, 1>, grid, block, stream, t);
    case 2: return launch_kernel(dequant_jobs_kernel<DT, 2>, grid, block, stream, t);
    case 4: return launch_kernel(dequant_jobs_kernel<DT, 4>, grid, block, stream, t);
    default: return hipErrorInvalidValue;
    }
}

template <int DT>
hipError_t launch_quant_anyshape_dt(int bits, int rounding, const QuantJob& a, hipStream_t stream) {
    return launch_kernel(quant_anyshape_kernel<DT>, dim3(a.grid_x, a.grid_y), dim3(kBlock), stream, a, bits,
                         rounding);
}

template <int DT>
hipError_t launch_dequant_anyshape_dt(const DequantJob& a, hipStream_t stream) {
    return launch_kernel(dequant_anyshape_kernel<DT>, dim3(a.grid_x, a.grid_y), dim3(kBlock), stream, a);
}

#define AQSGD_INSTANTIATE_DTYPE(DT)                                                               \
    template hipError_t launch_codec_jobs_dt<DT>(int, int, TableKind, const JobTable&, hipStream_t); \
    template hipError_t launch_dequant_jobs_dt<DT>(int, const JobTable&, hipStream_t);            \
    template hipError_t launch_quant_anyshape_dt<DT>(int, int, const QuantJob&, hipStream_t);     \
    template hipError_t launch_dequant_anyshape_dt<DT>(const DequantJob&, hipStream_t);

}  // namespace aqsgd
