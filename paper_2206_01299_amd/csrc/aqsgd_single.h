// Kernels of a launch that carries one message: encode, grad_quant, decode or grad_dequant
// called by itself.  The bodies are those of the shared launches (aqsgd_kernels.h); what
// differs is how a workgroup comes by its job.
//
// A launch of one micro-batch lasts 3 to 10 us, and the first microseconds pass before any
// of its data is asked for: the job is fetched from the argument buffer, the sample id
// through it, and only then the rows.  So the job is not a table here but a list of plain
// arguments whose first fourteen words (the pointers and what the addresses depend on) the
// hardware puts into scalar registers before a wave starts (the build asks for that with
// -amdgpu-kernarg-preload-count; structures are passed by reference and do not qualify).
// The workgroup's place is the grid's own x and y, and it does one step: what a loop would
// keep for the next one costs registers (loops around these bodies: 124 instead of 73) and
// with them waves in flight.  The arguments are 104 bytes (96 to reconstruct) where a table is 2000
// that the host copies for every launch.
// Measured, single calls as tables of one -> here: float16 [4,1024,1600] 4/8-bit, four calls
// 30.2 -> 27.9 us (20 us of it are the bytes); bfloat16 [32,256,1536] G = 64 3/6-bit, four
// calls 49.8 -> 46.8; first visits of half of that float16 batch 18.9 -> 17.6; 131072 float32
// elements, four calls, bound by the host's launches, 16.5 -> 13.9.
#pragma once

#include "aqsgd_kernels.h"

namespace aqsgd {

static_assert(sizeof(JobTable) == 2000, "the size named above");

// Words 0..13 are preloaded: five pointers, group, bits and n_per.
#define AQSGD_QUANT_ARGS                                                                                  \
    const void *src, const int64_t *ids, void *m_buf, uint8_t *codes, float *scales, int32_t group,       \
        int32_t bits, int64_t n_per, int64_t gps, int32_t batch, uint32_t grid_x, uint32_t grid_y,        \
        uint32_t stamp, uint64_t seed, uint32_t *seen, int32_t *first
#define AQSGD_DEQUANT_ARGS                                                                                \
    const uint8_t *codes, const float *scales, const int64_t *ids, void *m_buf, void *out, int32_t group, \
        int32_t bits, int64_t n_per, int64_t gps, int32_t batch, uint32_t grid_x, uint32_t grid_y,        \
        uint32_t stamp, uint32_t *seen, const void *full

// Which bodies a quantising kernel holds: as in the shared launches the 3-bit ones, which
// need more registers, are apart; odd groups have bodies of their own, and two kernels, for
// they have no table to go out with when a grid cannot hold one workgroup for every step.  The
// last kinds are the first two with m written through the L2 (see store16); they hold no bodies without m.
enum SingleKind { kSingleWhole = 0, kSingleThree, kSingleOdd, kSingleOddLoops, kSingleThrough, kSingleThreeThrough };

template <int DT, int BITS, int ROUND, int TEAM, int CPL, bool ODD, bool LOOPS, bool THROUGH = false>
__device__ __forceinline__ void single_quant_bits(const QuantJob& a, float* wave_max) {
    const uint32_t bx = blockIdx.x, by = blockIdx.y;
    if (THROUGH || a.m_buf) quant_team_body<DT, BITS, ROUND, TEAM, CPL, true, ODD, LOOPS, THROUGH>(a, bx, by, wave_max);
    else quant_team_body<DT, BITS, ROUND, TEAM, CPL, false, ODD, LOOPS, false>(a, bx, by, wave_max);
}

template <int DT, int ROUND, int TEAM, int CPL, int KIND>
__global__ __launch_bounds__((TEAM > kWave ? TEAM : kBlock))
void quant_single_kernel(AQSGD_QUANT_ARGS) {
    constexpr int kThreads = TEAM > kWave ? TEAM : kBlock;
    constexpr bool LOOPS = KIND == kSingleOddLoops;
    constexpr bool ODD = KIND == kSingleOdd || LOOPS;
    constexpr bool THROUGH = KIND == kSingleThrough || KIND == kSingleThreeThrough;
    [[maybe_unused]] __shared__ float wave_max[kThreads / kWave];
    QuantJob a;
    a.src = src; a.ids = ids; a.m_buf = m_buf; a.codes = codes; a.scales = scales;
    a.n_per = n_per; a.gps = gps; a.batch = batch; a.group = group; a.bits = bits;
    a.cpg = static_cast<int32_t>((static_cast<uint32_t>(group) + kChunk - 1) / kChunk);
    a.grid_x = grid_x; a.grid_y = grid_y; a.rcp_grid_x = 0.0f;
    a.seed = seed; a.seen = seen; a.first = first; a.stamp = stamp;
    if constexpr (KIND == kSingleThree || KIND == kSingleThreeThrough) {
        single_quant_bits<DT, 3, ROUND, TEAM, CPL, false, false, THROUGH>(a, wave_max);
    } else {
        switch (bits) {                                  // uniform over the launch
        case 2: single_quant_bits<DT, 2, ROUND, TEAM, CPL, ODD, LOOPS, THROUGH>(a, wave_max); break;
        case 4: single_quant_bits<DT, 4, ROUND, TEAM, CPL, ODD, LOOPS, THROUGH>(a, wave_max); break;
        case 6: single_quant_bits<DT, 6, ROUND, TEAM, CPL, ODD, LOOPS, THROUGH>(a, wave_max); break;
        default: single_quant_bits<DT, 8, ROUND, TEAM, CPL, ODD, LOOPS, THROUGH>(a, wave_max); break;
        }
    }
}

// THROUGH: how m and out are stored (see store16), a constant as in the shared launches.  Large
// reconstructions write through; the quantising side has kinds of its own for it (SingleKind).
template <int DT, int UNROLL, bool THROUGH>
__global__ __launch_bounds__(kBlock)
void dequant_single_kernel(AQSGD_DEQUANT_ARGS) {
    DequantJob a;
    a.codes = codes; a.scales = scales; a.ids = ids; a.m_buf = m_buf; a.out = out; a.full = full;
    a.n_per = n_per; a.gps = gps; a.cps = n_per >> 3; a.batch = batch; a.group = group;
    a.cpg = static_cast<int32_t>(static_cast<uint32_t>(group) / kChunk); a.bits = bits;
    a.grid_x = grid_x; a.grid_y = grid_y; a.rcp_grid_x = 0.0f;
    a.seen = seen; a.stamp = stamp;
    dequant_job<DT, UNROLL, kBlock, false, THROUGH>(a, blockIdx.x, blockIdx.y);
}

template <typename Kernel>
static hipError_t launch_quant_with(Kernel kernel, dim3 block, const QuantJob& a, hipStream_t s) {
    return launch_kernel(kernel, dim3(a.grid_x, a.grid_y), block, s, a.src, a.ids, a.m_buf, a.codes, a.scales,
                         a.group, a.bits, a.n_per, a.gps, a.batch, a.grid_x, a.grid_y, a.stamp, a.seed, a.seen,
                         a.first);
}

template <int DT, int ROUND, int TEAM, int CPL, int KIND>
static hipError_t launch_quant_single_as(const QuantJob& a, hipStream_t s) {
    return launch_quant_with(quant_single_kernel<DT, ROUND, TEAM, CPL, KIND>, dim3(TEAM > kWave ? TEAM : kBlock), a, s);
}

template <int DT, int ROUND, int KIND>
static hipError_t launch_quant_single_shape(int shape, const QuantJob& a, hipStream_t s) {
    switch (shape) {
    case kTeam2x1:
        if constexpr (KIND == kSingleOdd || KIND == kSingleOddLoops) return launch_quant_single_as<DT, ROUND, 2, 1, KIND>(a, s);
        else return hipErrorInvalidValue;
    case kTeam8x1:    return launch_quant_single_as<DT, ROUND, 8, 1, KIND>(a, s);
    case kTeam16x1:   return launch_quant_single_as<DT, ROUND, 16, 1, KIND>(a, s);
    case kTeam32x1:   return launch_quant_single_as<DT, ROUND, 32, 1, KIND>(a, s);
    case kTeam64x1:   return launch_quant_single_as<DT, ROUND, 64, 1, KIND>(a, s);
    case kTeam64x2:   return launch_quant_single_as<DT, ROUND, 64, 2, KIND>(a, s);
    case kTeam64x3:   return launch_quant_single_as<DT, ROUND, 64, 3, KIND>(a, s);
    case kTeam64x4:   return launch_quant_single_as<DT, ROUND, 64, 4, KIND>(a, s);
    case kTeam256x2:  return launch_quant_single_as<DT, ROUND, 256, 2, KIND>(a, s);
    case kTeam256x4:  return launch_quant_single_as<DT, ROUND, 256, 4, KIND>(a, s);
    case kTeam1024x2: return launch_quant_single_as<DT, ROUND, 1024, 2, KIND>(a, s);
    case kTeam1024x4: return launch_quant_single_as<DT, ROUND, 1024, 4, KIND>(a, s);
    default:          return hipErrorInvalidValue;
    }
}

template <int DT, int ROUND>
static hipError_t launch_quant_single_kind(int shape, bool covers, bool through, const QuantJob& a, hipStream_t s) {
    if (!covers && a.group % kChunk != 0) return launch_quant_single_shape<DT, ROUND, kSingleOddLoops>(shape, a, s);
    if (!covers) return hipErrorInvalidValue;
    if (a.group % kChunk != 0) return launch_quant_single_shape<DT, ROUND, kSingleOdd>(shape, a, s);
    if (through && a.m_buf)
        return a.bits == 3 ? launch_quant_single_shape<DT, ROUND, kSingleThreeThrough>(shape, a, s)
                           : launch_quant_single_shape<DT, ROUND, kSingleThrough>(shape, a, s);
    if (a.bits == 3) return launch_quant_single_shape<DT, ROUND, kSingleThree>(shape, a, s);
    return launch_quant_single_shape<DT, ROUND, kSingleWhole>(shape, a, s);
}

// `covers`: the job's rectangle has a workgroup for every sample and step; `through`: how m is stored.
template <int DT>
hipError_t launch_quant_single_dt(int rounding, int shape, bool covers, bool through, const QuantJob& a, hipStream_t s) {
    return rounding == AQSGD_ROUND_STOCHASTIC
               ? launch_quant_single_kind<DT, AQSGD_ROUND_STOCHASTIC>(shape, covers, through, a, s)
               : launch_quant_single_kind<DT, AQSGD_ROUND_NEAREST>(shape, covers, through, a, s);
}

template <typename Kernel>
static hipError_t launch_dequant_with(Kernel kernel, const DequantJob& a, hipStream_t s) {
    return launch_kernel(kernel, dim3(a.grid_x, a.grid_y), dim3(kBlock), s, a.codes, a.scales, a.ids, a.m_buf, a.out,
                         a.group, a.bits, a.n_per, a.gps, a.batch, a.grid_x, a.grid_y, a.stamp, a.seen, a.full);
}

template <int DT, bool THROUGH>
static hipError_t launch_dequant_single_unroll(int unroll, const DequantJob& a, hipStream_t s) {
    switch (unroll) {
    case 1: return launch_dequant_with(dequant_single_kernel<DT, 1, THROUGH>, a, s);
    case 2: return launch_dequant_with(dequant_single_kernel<DT, 2, THROUGH>, a, s);
    case 4: return launch_dequant_with(dequant_single_kernel<DT, 4, THROUGH>, a, s);
    default: return hipErrorInvalidValue;
    }
}

template <int DT>
hipError_t launch_dequant_single_dt(int unroll, bool through, const DequantJob& a, hipStream_t s) {
    return through ? launch_dequant_single_unroll<DT, true>(unroll, a, s)
                   : launch_dequant_single_unroll<DT, false>(unroll, a, s);
}

#define AQSGD_INSTANTIATE_SINGLE_DTYPE(DT)                                                        \
    template hipError_t launch_quant_single_dt<DT>(int, int, bool, bool, const QuantJob&, hipStream_t); \
    template hipError_t launch_dequant_single_dt<DT>(int, bool, const DequantJob&, hipStream_t);

}  // namespace aqsgd
