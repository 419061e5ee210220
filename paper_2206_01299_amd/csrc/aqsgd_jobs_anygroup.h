// Shared launches of messages outside the job kernels' range (aqsgd_kernels.h): the quantising
// jobs are odd groups of one team shape, or wide groups, and the dequantising jobs that are ready
// with them go along, all behind the same job table.  Each such message used to have launches of
// its own, and a time slot of a stage boundary is four messages a boundary, none of them large
// enough to fill the chip: an odd-group message of half a megabyte lasts 3 to 5 us whatever it
// holds, and a group of 50000 elements keeps one compute unit busy for 5 to 20 us while the others
// have nothing to do.
//
// Measured, a message a launch -> shared, a time slot (four messages) of one boundary: float16
// [6,75,580], rows of 580 14.1 -> 5.9 us (four boundaries 60.2 -> 10.1), [4,250,1020] 15.1 -> 7.6;
// one scale per sample, float16 [8,64,768] 19.3 -> 9.8, stochastic 19.0 -> 9.5; bfloat16 [29,339,104]
// stochastic, three boundaries 60.6 -> 18.9 (54 MB).
#pragma once

#include "aqsgd_anygroup.h"

namespace aqsgd {

// This workgroup's job and its place in the job's rectangle (as in codec_jobs_kernel).  Everything
// in here has to be inlined into the kernel: a call that takes a job by its address makes the
// compiler copy the whole table to every lane's scratch memory, 2 KB a lane, more than the chip can
// give a workgroup of 1024 lanes, which then never starts.
#define AQSGD_INLINE __attribute__((always_inline))
template <typename Quant, typename Dequant>
__device__ __forceinline__ void run_table_job(const JobTable& t, Quant&& quant, Dequant&& dequant) {
    const uint32_t b = blockIdx.x;
    touch_lines(&t, 0, 63);
    touch_lines(&t, offsetof(JobTable, q), offsetof(JobTable, q) + sizeof(QuantJob) - 1);
    uint32_t bx, by;
    if (b < t.dequant_block0) {
        const BlockStarts qs = block_starts(t.q_block0);
        const int j = job_of_block(qs, t.n_quant, b);
        const QuantJob& a = t.q[j];
        place_in_job(b - start_of_job(qs, j), a.grid_x, a.rcp_grid_x, bx, by);
        quant(a, bx, by);
    } else {
        const BlockStarts ds = block_starts(t.d_block0);
        const int j = job_of_block(ds, t.n_dequant, b);
        const DequantJob& a = t.d[j];
        place_in_job(b - start_of_job(ds, j), a.grid_x, a.rcp_grid_x, bx, by);
        dequant(a, bx, by);
    }
}

// Odd groups of one rounding mode and team shape, any odd dequantising jobs; a workgroup for
// every step of every sample.
template <int DT, int ROUND, int TEAM, int CPL>
__global__ __launch_bounds__((TEAM > kWave ? TEAM : kBlock))
void odd_jobs_kernel(const JobTable t) {
    constexpr int kThreads = TEAM > kWave ? TEAM : kBlock;
    [[maybe_unused]] __shared__ float wave_max[kThreads / kWave];
    run_table_job(t,
        [&](const QuantJob& a, uint32_t bx, uint32_t by) AQSGD_INLINE {
            auto body = [&](auto bits) AQSGD_INLINE {
                constexpr int BITS = decltype(bits)::value;
                if (a.m_buf) quant_team_body<DT, BITS, ROUND, TEAM, CPL, true, true, false, false>(a, bx, by, wave_max);
                else quant_team_body<DT, BITS, ROUND, TEAM, CPL, false, true, false, false>(a, bx, by, wave_max);
            };
            switch (a.bits) {                            // uniform over the workgroup
            case 2: body(std::integral_constant<int, 2>()); break;
            case 4: body(std::integral_constant<int, 4>()); break;
            case 6: body(std::integral_constant<int, 6>()); break;
            default: body(std::integral_constant<int, 8>()); break;
            }
        },
        [&](const DequantJob& a, uint32_t bx, uint32_t by) AQSGD_INLINE { dequant_odd_job<DT, kThreads, false>(a, bx, by); });
}

// Wide groups, one workgroup each, and dequantising jobs of whole chunks.
template <int DT, int ROUND>
__global__ __launch_bounds__(kWideThreads)
void wide_jobs_kernel(const JobTable t) {
    __shared__ float wave_max[kWideThreads / kWave];
    run_table_job(t,
        [&](const QuantJob& a, uint32_t bx, uint32_t by) AQSGD_INLINE { quant_wide_job<DT, ROUND>(a, bx, by, 0, 1 << 20, wave_max); },
        [&](const DequantJob& a, uint32_t bx, uint32_t by) AQSGD_INLINE {
            dequant_job<DT, kHostedDequantUnroll, kWideThreads, false, false>(a, bx, by);
        });
}

// Few wide groups, split into spans: the maxima of all jobs, then the levels and the dequantising jobs.
template <int DT>
__global__ __launch_bounds__(kBlock)
void split_max_jobs_kernel(const JobTable t) {
    __shared__ float wave_max[kBlock / kWave];
    run_table_job(t,
        [&](const QuantJob& a, uint32_t bx, uint32_t by) AQSGD_INLINE {
            split_max_job<DT>(a, split_geometry(a), Rect{bx, by, a.grid_x, a.grid_y}, wave_max);
        },
        [](const DequantJob&, uint32_t, uint32_t) AQSGD_INLINE {});
}
template <int DT, int ROUND>
__global__ __launch_bounds__(kBlock)
void split_jobs_kernel(const JobTable t) {
    run_table_job(t,
        [&](const QuantJob& a, uint32_t bx, uint32_t by) AQSGD_INLINE {
            split_quant_job<DT, ROUND>(a, split_geometry(a), Rect{bx, by, a.grid_x, a.grid_y});
        },
        [&](const DequantJob& a, uint32_t bx, uint32_t by) AQSGD_INLINE {
            dequant_job<DT, kHostedDequantUnroll, kBlock, false, false>(a, bx, by);
        });
}

// Per-dtype pieces (defined by AQSGD_INSTANTIATE_JOBS_ANYGROUP_DTYPE in the dtype's .hip file).
template <int DT> hipError_t launch_odd_jobs_dt(int rounding, int shape, const JobTable& t, hipStream_t stream);
template <int DT> hipError_t launch_wide_jobs_dt(int rounding, const JobTable& t, hipStream_t stream);
template <int DT> hipError_t launch_split_jobs_dt(int rounding, const JobTable& t, hipStream_t stream);

// ---- launch tables (instantiated per dtype in aqsgd_jobs_anygroup_<dtype>.hip) ----------
template <int DT, int ROUND, int TEAM, int CPL>
static hipError_t launch_oj(const JobTable& t, hipStream_t s) {
    return launch_kernel(odd_jobs_kernel<DT, ROUND, TEAM, CPL>, dim3(t.total_blocks),
                         dim3(TEAM > kWave ? TEAM : kBlock), s, t);
}

template <int DT, int ROUND>
static hipError_t launch_oj_shape(int shape, const JobTable& t, hipStream_t s) {
    switch (shape) {
    case kTeam2x1:    return launch_oj<DT, ROUND, 2, 1>(t, s);
    case kTeam8x1:    return launch_oj<DT, ROUND, 8, 1>(t, s);
    case kTeam16x1:   return launch_oj<DT, ROUND, 16, 1>(t, s);
    case kTeam32x1:   return launch_oj<DT, ROUND, 32, 1>(t, s);
    case kTeam64x1:   return launch_oj<DT, ROUND, 64, 1>(t, s);
    case kTeam64x2:   return launch_oj<DT, ROUND, 64, 2>(t, s);
    case kTeam64x3:   return launch_oj<DT, ROUND, 64, 3>(t, s);
    case kTeam64x4:   return launch_oj<DT, ROUND, 64, 4>(t, s);
    case kTeam256x2:  return launch_oj<DT, ROUND, 256, 2>(t, s);
    case kTeam256x4:  return launch_oj<DT, ROUND, 256, 4>(t, s);
    case kTeam1024x2: return launch_oj<DT, ROUND, 1024, 2>(t, s);
    case kTeam1024x4: return launch_oj<DT, ROUND, 1024, 4>(t, s);
    default:          return hipErrorInvalidValue;
    }
}

template <int DT>
hipError_t launch_odd_jobs_dt(int rounding, int shape, const JobTable& t, hipStream_t s) {
    return rounding == AQSGD_ROUND_STOCHASTIC ? launch_oj_shape<DT, AQSGD_ROUND_STOCHASTIC>(shape, t, s)
                                              : launch_oj_shape<DT, AQSGD_ROUND_NEAREST>(shape, t, s);
}

template <int DT>
hipError_t launch_wide_jobs_dt(int rounding, const JobTable& t, hipStream_t s) {
    const dim3 grid(t.total_blocks), block(kWideThreads);
    return rounding == AQSGD_ROUND_STOCHASTIC
               ? launch_kernel(wide_jobs_kernel<DT, AQSGD_ROUND_STOCHASTIC>, grid, block, s, t)
               : launch_kernel(wide_jobs_kernel<DT, AQSGD_ROUND_NEAREST>, grid, block, s, t);
}

template <int DT>
hipError_t launch_split_jobs_dt(int rounding, const JobTable& t, hipStream_t s) {
    const dim3 grid(t.total_blocks), block(kBlock);
    ProfileSpan span;
    // the quantising jobs' workgroups come first in a table
    const hipError_t err = launch_kernel(split_max_jobs_kernel<DT>, dim3(t.dequant_block0), block, s, t);
    if (err != hipSuccess) return err;
    span.last();
    return rounding == AQSGD_ROUND_STOCHASTIC
               ? launch_kernel(split_jobs_kernel<DT, AQSGD_ROUND_STOCHASTIC>, grid, block, s, t)
               : launch_kernel(split_jobs_kernel<DT, AQSGD_ROUND_NEAREST>, grid, block, s, t);
}

#define AQSGD_INSTANTIATE_JOBS_ANYGROUP_DTYPE(DT)                                               \
    template hipError_t launch_odd_jobs_dt<DT>(int, int, const JobTable&, hipStream_t);         \
    template hipError_t launch_wide_jobs_dt<DT>(int, const JobTable&, hipStream_t);             \
    template hipError_t launch_split_jobs_dt<DT>(int, const JobTable&, hipStream_t);

#undef AQSGD_INLINE

}  // namespace aqsgd
