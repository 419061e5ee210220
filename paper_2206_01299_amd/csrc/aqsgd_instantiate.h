// Launch tables of one storage dtype: every (rounding, team shape, kind) of the job
// kernel that hosts quantising jobs and every unroll of the one that holds
// dequantising jobs alone.  Each dtype gets a translation unit for the kernels that stream
// and one for those that write through, so that they compile in parallel.
#pragma once

#include "aqsgd_kernels.h"

namespace aqsgd {

template <int DT, int ROUND, int KIND, bool THROUGH, int TEAM, int CPL>
static hipError_t launch_cj(const JobTable& t, hipStream_t stream) {
    constexpr int threads = TEAM > kWave ? TEAM : kBlock;
    // Teams of a wavefront and more loop only where a cap on the grid asks for it: one kernel does.
    // It streams, too: launches of that size or number of samples are rare and the kernel the largest.
    if constexpr (THROUGH && (KIND == kTableLoops || KIND == kTableLoopsThree) && TEAM >= kWave) return hipErrorInvalidValue;
    else if constexpr (KIND == kTableLoops && TEAM >= kWave)
        return launch_cj<DT, ROUND, kTableLoopsThree, THROUGH, TEAM, CPL>(t, stream);
    else return launch_kernel(codec_jobs_kernel<DT, ROUND, TEAM, CPL, KIND, THROUGH>, dim3(t.total_blocks), dim3(threads),
                              stream, t);
}

template <int DT, int ROUND, int KIND, bool THROUGH>
static hipError_t launch_cj_shape(int shape, const JobTable& t, hipStream_t stream) {
    switch (shape) {
    case kTeam8x1:    return launch_cj<DT, ROUND, KIND, THROUGH, 8, 1>(t, stream);
    case kTeam16x1:   return launch_cj<DT, ROUND, KIND, THROUGH, 16, 1>(t, stream);
    case kTeam32x1:   return launch_cj<DT, ROUND, KIND, THROUGH, 32, 1>(t, stream);
    case kTeam64x1:   return launch_cj<DT, ROUND, KIND, THROUGH, 64, 1>(t, stream);
    case kTeam64x2:   return launch_cj<DT, ROUND, KIND, THROUGH, 64, 2>(t, stream);
    case kTeam64x3:   return launch_cj<DT, ROUND, KIND, THROUGH, 64, 3>(t, stream);
    case kTeam64x4:   return launch_cj<DT, ROUND, KIND, THROUGH, 64, 4>(t, stream);
    case kTeam256x2:  return launch_cj<DT, ROUND, KIND, THROUGH, 256, 2>(t, stream);
    case kTeam256x4:  return launch_cj<DT, ROUND, KIND, THROUGH, 256, 4>(t, stream);
    case kTeam1024x2: return launch_cj<DT, ROUND, KIND, THROUGH, 1024, 2>(t, stream);
    case kTeam1024x4: return launch_cj<DT, ROUND, KIND, THROUGH, 1024, 4>(t, stream);
    default:          return hipErrorInvalidValue;
    }
}

template <int DT, int ROUND, bool THROUGH>
static hipError_t launch_cj_kind(int shape, TableKind kind, const JobTable& t, hipStream_t stream) {
    switch (kind) {
    case kTableOneStep:      return launch_cj_shape<DT, ROUND, kTableOneStep, THROUGH>(shape, t, stream);
    case kTableOneStepThree: return launch_cj_shape<DT, ROUND, kTableOneStepThree, THROUGH>(shape, t, stream);
    case kTableLoops:        return launch_cj_shape<DT, ROUND, kTableLoops, THROUGH>(shape, t, stream);
    case kTableLoopsThree:   return launch_cj_shape<DT, ROUND, kTableLoopsThree, THROUGH>(shape, t, stream);
    default:                 return hipErrorInvalidValue;
    }
}

template <int DT, bool THROUGH>
hipError_t launch_codec_jobs_dt(int rounding, int shape, TableKind kind, const JobTable& t, hipStream_t stream) {
    return rounding == AQSGD_ROUND_STOCHASTIC
               ? launch_cj_kind<DT, AQSGD_ROUND_STOCHASTIC, THROUGH>(shape, kind, t, stream)
               : launch_cj_kind<DT, AQSGD_ROUND_NEAREST, THROUGH>(shape, kind, t, stream);
}

template <int DT, bool THROUGH>
hipError_t launch_dequant_jobs_dt(int unroll, const JobTable& t, hipStream_t stream) {
    const dim3 grid(t.total_blocks), block(kBlock);
    switch (unroll) {
    case 1: return launch_kernel(dequant_jobs_kernel<DT, 1, THROUGH>, grid, block, stream, t);
    case 2: return launch_kernel(dequant_jobs_kernel<DT, 2, THROUGH>, grid, block, stream, t);
    case 4: return launch_kernel(dequant_jobs_kernel<DT, 4, THROUGH>, grid, block, stream, t);
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

#define AQSGD_INSTANTIATE_TABLES(DT, THROUGH)                                                     \
    template hipError_t launch_codec_jobs_dt<DT, THROUGH>(int, int, TableKind, const JobTable&, hipStream_t); \
    template hipError_t launch_dequant_jobs_dt<DT, THROUGH>(int, const JobTable&, hipStream_t);
#define AQSGD_INSTANTIATE_DTYPE(DT)                                                               \
    AQSGD_INSTANTIATE_TABLES(DT, false)                                                           \
    template hipError_t launch_quant_anyshape_dt<DT>(int, int, const QuantJob&, hipStream_t);     \
    template hipError_t launch_dequant_anyshape_dt<DT>(const DequantJob&, hipStream_t);

}  // namespace aqsgd
