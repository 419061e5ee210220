// C ABI of the AQ-SGD boundary codec: argument checks and kernel dispatch.
// See include/aqsgd.h for the contract of every entry point.
#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <limits>
#include <type_traits>
#include <vector>

#include "aqsgd_anygroup.h"
#include "aqsgd_jobs_anygroup.h"
#include "aqsgd_kernels.h"
#include "aqsgd_lowbit.h"
#include "aqsgd_single.h"
#include "aqsgd_topk.h"
#include "aqsgd_topk_small.h"

namespace aqsgd {

// Instantiated in the dtypes' own translation units.
#define AQSGD_EXTERN_DTYPE(DT)                                                                        \
    extern template hipError_t launch_quant_single_dt<DT>(int, int, bool, bool, const QuantJob&, hipStream_t); \
    extern template hipError_t launch_dequant_single_dt<DT>(int, bool, const DequantJob&, hipStream_t); \
    extern template hipError_t launch_dequant_odd_dt<DT>(bool, bool, const DequantJob&, hipStream_t); \
    extern template hipError_t launch_quant_wide_dt<DT>(int, int, int, const QuantJob&, hipStream_t); \
    extern template hipError_t launch_quant_large_dt<DT>(int, const QuantJob&, const LargeGeom&, hipStream_t); \
    extern template hipError_t launch_quant_split_dt<DT>(int, const QuantJob&, const LargeGeom&, hipStream_t); \
    extern template hipError_t launch_odd_jobs_dt<DT>(int, int, const JobTable&, hipStream_t);        \
    extern template hipError_t launch_wide_jobs_dt<DT>(int, const JobTable&, hipStream_t);            \
    extern template hipError_t launch_split_jobs_dt<DT>(int, const JobTable&, hipStream_t);           \
    extern template hipError_t launch_lowbit_dt<DT>(int, int, int, bool, LaunchGeom, const LowbitArgs&, hipStream_t);
AQSGD_EXTERN_DTYPE(AQSGD_F32)
AQSGD_EXTERN_DTYPE(AQSGD_F16)
AQSGD_EXTERN_DTYPE(AQSGD_BF16)

thread_local ProfileRequest g_profile_request = {nullptr, nullptr};

// -- dtype fan-out (each dtype's kernels live in their own translation unit) ----
template <bool THROUGH>
hipError_t launch_codec_jobs_as(int dtype, int rounding, int shape, TableKind kind, const JobTable& t, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_codec_jobs_dt<AQSGD_F32, THROUGH>(rounding, shape, kind, t, s);
    case AQSGD_F16:  return launch_codec_jobs_dt<AQSGD_F16, THROUGH>(rounding, shape, kind, t, s);
    case AQSGD_BF16: return launch_codec_jobs_dt<AQSGD_BF16, THROUGH>(rounding, shape, kind, t, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_codec_jobs(int dtype, int rounding, int shape, TableKind kind, bool through, const JobTable& t,
                             hipStream_t s) {
    return through ? launch_codec_jobs_as<true>(dtype, rounding, shape, kind, t, s)
                   : launch_codec_jobs_as<false>(dtype, rounding, shape, kind, t, s);
}
template <bool THROUGH>
hipError_t launch_dequant_jobs_as(int dtype, int unroll, const JobTable& t, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_dequant_jobs_dt<AQSGD_F32, THROUGH>(unroll, t, s);
    case AQSGD_F16:  return launch_dequant_jobs_dt<AQSGD_F16, THROUGH>(unroll, t, s);
    case AQSGD_BF16: return launch_dequant_jobs_dt<AQSGD_BF16, THROUGH>(unroll, t, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_dequant_jobs(int dtype, int unroll, bool through, const JobTable& t, hipStream_t s) {
    return through ? launch_dequant_jobs_as<true>(dtype, unroll, t, s) : launch_dequant_jobs_as<false>(dtype, unroll, t, s);
}
hipError_t launch_quant_anyshape(int dtype, int bits, int rounding, const QuantJob& a, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_quant_anyshape_dt<AQSGD_F32>(bits, rounding, a, s);
    case AQSGD_F16:  return launch_quant_anyshape_dt<AQSGD_F16>(bits, rounding, a, s);
    case AQSGD_BF16: return launch_quant_anyshape_dt<AQSGD_BF16>(bits, rounding, a, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_dequant_anyshape(int dtype, const DequantJob& a, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_dequant_anyshape_dt<AQSGD_F32>(a, s);
    case AQSGD_F16:  return launch_dequant_anyshape_dt<AQSGD_F16>(a, s);
    case AQSGD_BF16: return launch_dequant_anyshape_dt<AQSGD_BF16>(a, s);
    default:         return hipErrorInvalidValue;
    }
}

hipError_t launch_quant_single(int dtype, int rounding, int shape, bool covers, bool through, const QuantJob& a,
                               hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_quant_single_dt<AQSGD_F32>(rounding, shape, covers, through, a, s);
    case AQSGD_F16:  return launch_quant_single_dt<AQSGD_F16>(rounding, shape, covers, through, a, s);
    case AQSGD_BF16: return launch_quant_single_dt<AQSGD_BF16>(rounding, shape, covers, through, a, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_dequant_single(int dtype, int unroll, bool through, const DequantJob& a, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_dequant_single_dt<AQSGD_F32>(unroll, through, a, s);
    case AQSGD_F16:  return launch_dequant_single_dt<AQSGD_F16>(unroll, through, a, s);
    case AQSGD_BF16: return launch_dequant_single_dt<AQSGD_BF16>(unroll, through, a, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_dequant_odd(int dtype, bool covers, bool through, const DequantJob& a, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_dequant_odd_dt<AQSGD_F32>(covers, through, a, s);
    case AQSGD_F16:  return launch_dequant_odd_dt<AQSGD_F16>(covers, through, a, s);
    case AQSGD_BF16: return launch_dequant_odd_dt<AQSGD_BF16>(covers, through, a, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_quant_wide(int dtype, int rounding, int parts, int share, const QuantJob& a, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_quant_wide_dt<AQSGD_F32>(rounding, parts, share, a, s);
    case AQSGD_F16:  return launch_quant_wide_dt<AQSGD_F16>(rounding, parts, share, a, s);
    case AQSGD_BF16: return launch_quant_wide_dt<AQSGD_BF16>(rounding, parts, share, a, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_quant_large(int dtype, int rounding, const QuantJob& a, const LargeGeom& geom, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_quant_large_dt<AQSGD_F32>(rounding, a, geom, s);
    case AQSGD_F16:  return launch_quant_large_dt<AQSGD_F16>(rounding, a, geom, s);
    case AQSGD_BF16: return launch_quant_large_dt<AQSGD_BF16>(rounding, a, geom, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_quant_split(int dtype, int rounding, const QuantJob& a, const LargeGeom& geom, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_quant_split_dt<AQSGD_F32>(rounding, a, geom, s);
    case AQSGD_F16:  return launch_quant_split_dt<AQSGD_F16>(rounding, a, geom, s);
    case AQSGD_BF16: return launch_quant_split_dt<AQSGD_BF16>(rounding, a, geom, s);
    default:         return hipErrorInvalidValue;
    }
}

hipError_t launch_odd_jobs(int dtype, int rounding, int shape, const JobTable& t, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_odd_jobs_dt<AQSGD_F32>(rounding, shape, t, s);
    case AQSGD_F16:  return launch_odd_jobs_dt<AQSGD_F16>(rounding, shape, t, s);
    case AQSGD_BF16: return launch_odd_jobs_dt<AQSGD_BF16>(rounding, shape, t, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_wide_jobs(int dtype, int rounding, const JobTable& t, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_wide_jobs_dt<AQSGD_F32>(rounding, t, s);
    case AQSGD_F16:  return launch_wide_jobs_dt<AQSGD_F16>(rounding, t, s);
    case AQSGD_BF16: return launch_wide_jobs_dt<AQSGD_BF16>(rounding, t, s);
    default:         return hipErrorInvalidValue;
    }
}
hipError_t launch_split_jobs(int dtype, int rounding, const JobTable& t, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_split_jobs_dt<AQSGD_F32>(rounding, t, s);
    case AQSGD_F16:  return launch_split_jobs_dt<AQSGD_F16>(rounding, t, s);
    case AQSGD_BF16: return launch_split_jobs_dt<AQSGD_BF16>(rounding, t, s);
    default:         return hipErrorInvalidValue;
    }
}

hipError_t launch_lowbit(int dtype, int bits, int m_bits, int shape, bool sender, LaunchGeom g,
                         const LowbitArgs& a, hipStream_t s) {
    switch (dtype) {
    case AQSGD_F32:  return launch_lowbit_dt<AQSGD_F32>(bits, m_bits, shape, sender, g, a, s);
    case AQSGD_F16:  return launch_lowbit_dt<AQSGD_F16>(bits, m_bits, shape, sender, g, a, s);
    case AQSGD_BF16: return launch_lowbit_dt<AQSGD_BF16>(bits, m_bits, shape, sender, g, a, s);
    default:         return hipErrorInvalidValue;
    }
}

namespace {

// Launch-shape knobs.  They change how the work is cut into workgroups, never a
// result bit.  Defaults come from the environment, once, so a sweep needs no
// rebuild; aqsgd_set_launch_shape overrides them for the process.  Each knob is
// an atomic of its own: a call reads each one once, so a change made by another
// thread takes effect for whole calls only.
int env_int(const char* name, int fallback) {
    const char* v = std::getenv(name);
    if (!v || !*v) return fallback;
    char* end = nullptr;
    const long x = std::strtol(v, &end, 10);
    return (end && *end == '\0' && x > 0 && x < (1L << 30)) ? static_cast<int>(x) : fallback;
}

int64_t env_max_blocks() { return env_int("AQSGD_MAX_BLOCKS", 1 << 20); }
int env_dequant_unroll() {
    const int u = env_int("AQSGD_DEQUANT_UNROLL", 2);
    return (u == 1 || u == 2 || u == 4) ? u : 2;
}

std::atomic<int64_t>& max_blocks_knob() {
    static std::atomic<int64_t> v{env_max_blocks()};
    return v;
}
std::atomic<int>& dequant_unroll_knob() {
    static std::atomic<int> v{env_dequant_unroll()};
    return v;
}

// Workgroups per launch that carries several jobs; 0 = the library's own choice (see
// steps_per_workgroup).  For sweeps only: AQSGD_LAUNCH_BLOCKS in the environment.
int64_t env_launch_blocks() { return env_int("AQSGD_LAUNCH_BLOCKS", 0); }
std::atomic<int64_t>& launch_blocks_knob() {
    static std::atomic<int64_t> v{env_launch_blocks()};
    return v;
}

constexpr int64_t kMaxGridY = 65535;
constexpr int kMaxTeamChunks = 4096;     // 1024 lanes x 4 chunks x 8 elements = 32768 elements

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

int check_desc(const aqsgd_desc* d, bool needs_buffer) {
    if (!d) return AQSGD_ERR_NULL;
    if (d->dtype != AQSGD_F32 && d->dtype != AQSGD_F16 && d->dtype != AQSGD_BF16) return AQSGD_ERR_DTYPE;
    if (d->rounding != AQSGD_ROUND_NEAREST && d->rounding != AQSGD_ROUND_STOCHASTIC) return AQSGD_ERR_DTYPE;
    if (!(d->bits == 2 || d->bits == 3 || d->bits == 4 || d->bits == 6 || d->bits == 8)) return AQSGD_ERR_BITS;
    if (d->batch < 0 || d->n_per <= 0) return AQSGD_ERR_SHAPE;
    if (d->group <= 0 || d->n_per % d->group != 0) return AQSGD_ERR_GROUP;
    if ((static_cast<int64_t>(d->group) * d->bits) % 8 != 0) return AQSGD_ERR_GROUP;
    const int64_t lim = std::numeric_limits<int64_t>::max() / 16;
    if (d->batch > std::numeric_limits<int32_t>::max()) return AQSGD_ERR_SHAPE;
    if (d->n_per > (int64_t{1} << 34)) return AQSGD_ERR_SHAPE;            // chunk index fits 32 bits
    if (d->batch > 0 && d->n_per > lim / d->batch) return AQSGD_ERR_SHAPE;
    if (needs_buffer) {
        if (d->n_samples <= 0 || d->n_per > lim / d->n_samples) return AQSGD_ERR_SHAPE;
    }
    return AQSGD_OK;
}

int team_shape_for(int cpg) {
    if (cpg <= 8) return kTeam8x1;
    if (cpg <= 16) return kTeam16x1;
    if (cpg <= 32) return kTeam32x1;
    if (cpg <= 64) return kTeam64x1;
    if (cpg <= 128) return kTeam64x2;
    if (cpg <= 192) return kTeam64x3;
    if (cpg <= 256) return kTeam64x4;
    if (cpg <= 512) return kTeam256x2;
    if (cpg <= 1024) return kTeam256x4;
    if (cpg <= 2048) return kTeam1024x2;
    return kTeam1024x4;
}

// Odd groups of two chunks (9 to 15 elements) have a team of two lanes: in a team of eight, six lanes
// repeat the last chunk, draw its random numbers and store its results once more.  Measured on 4 M
// elements, eight lanes -> two (one thread per group): stochastic grad_quant, groups of 9 at 8 bits,
// float16 24.7 -> 9.1 us (14.5), float32 29.9 -> 10.8 (16.2), of 14 at 4 bits 17.2 -> 6.8 (14.7) and
// 20.8 -> 7.6 (19.4); float16 encode, groups of 9, nearest 24.8 -> 10.5 (22.3).  Nearest encode in
// float32 keeps eight: groups of 12 at 4 bits 16.4 us, with two lanes 19.6 (50.8; of 9 at 8 bits
// 25.1 and 20.1).
int odd_team_shape_for(int cpg, int dtype, int rounding, bool has_buf) {
    const bool eight = dtype == AQSGD_F32 && has_buf && rounding == AQSGD_ROUND_NEAREST;
    return cpg <= 2 && !eight ? static_cast<int>(kTeam2x1) : team_shape_for(cpg);
}

// Groups one step of a workgroup of the quantising kernel covers (its teams times the
// groups each takes, groups_per_team).
int groups_per_block_step(int shape) {
    switch (shape) {
    case kTeam2x1: return kBlock / 2 * groups_per_team(2, 1);
    case kTeam8x1: return kBlock / 8 * groups_per_team(8, 1);
    case kTeam16x1: return kBlock / 16 * groups_per_team(16, 1);
    case kTeam32x1: return kBlock / 32 * groups_per_team(32, 1);
    case kTeam64x1: return kBlock / 64 * groups_per_team(64, 1);
    case kTeam64x2: case kTeam64x3: case kTeam64x4: return kBlock / 64;
    default: return 1;
    }
}

// Workgroups of one job: grid_y walks the samples, grid_x the pieces of a sample,
// bounded by `max_blocks` in all (the kernels loop over what is left).
LaunchGeom geometry(int64_t units_per_sample, int64_t units_per_block, int64_t batch, int64_t max_blocks) {
    LaunchGeom g;
    const int64_t gy = batch < kMaxGridY ? batch : kMaxGridY;
    int64_t gx = (units_per_sample + units_per_block - 1) / units_per_block;
    const int64_t cap = max_blocks / gy > 0 ? max_blocks / gy : 1;
    if (gx > cap) gx = cap;
    if (gx < 1) gx = 1;
    g.grid_x = static_cast<uint32_t>(gx);
    g.grid_y = static_cast<uint32_t>(gy);
    return g;
}

int threads_of_shape(int shape) {
    switch (shape) {
    case kTeam1024x2: case kTeam1024x4: return 1024;
    default: return kBlock;
    }
}

// First-visit arguments of the *_seen entry points (all null / 0 otherwise).
struct SeenArgs {
    uint32_t* seen = nullptr;
    int32_t* first = nullptr;
    const void* full = nullptr;
    uint32_t stamp = 0;
};

// Pieces of 16 bytes (the dequantising side's unit for odd groups) of a sample.
int64_t odd_pieces(const DequantJob& a, int dtype) {
    const int64_t piece = dtype == AQSGD_F32 ? kUnit : kChunk;
    return (a.n_per + piece - 1) / piece;
}

// Which kernels a message takes.  Groups of whole chunks that fit a workgroup's registers are
// jobs of the shared launches; odd groups (8 elements or more, not whole chunks) and groups beyond the
// job kernels' team shapes share launches of their own.  Launched one by one: groups beyond any
// workgroup (quantising side only: reconstruction needs no maximum), and those of 1 to 7 elements, which
// have no 16-byte piece and take the scalar kernels.
enum class Route { kJob, kOdd, kWide, kLarge, kAnyShape };

// One message as the kernels see it.  Quantising side: aqsgd_encode, aqsgd_grad_quant.
struct QuantPlan {
    QuantJob job;
    int dtype, bits, rounding;
    Route route;
    int shape;                 // team shape (kJob, kOdd)
};

QuantPlan plan_quant(const aqsgd_desc* d, int64_t batch, int64_t n_per, const void* src, const int64_t* ids,
                     void* m_buf, uint8_t* codes, float* scales, const SeenArgs& sa = SeenArgs()) {
    QuantPlan p;
    QuantJob& a = p.job;
    a.src = src; a.ids = ids; a.m_buf = m_buf; a.codes = codes; a.scales = scales;
    a.n_per = n_per; a.gps = n_per / d->group;
    a.batch = static_cast<int32_t>(batch); a.group = d->group; a.bits = d->bits;
    a.cpg = static_cast<int32_t>((static_cast<int64_t>(d->group) + kChunk - 1) / kChunk);
    a.grid_x = a.grid_y = 1; a.rcp_grid_x = 1.0f;
    a.seed = d->rng_seed; a.seen = sa.seen; a.first = sa.first; a.stamp = sa.stamp;
    p.dtype = d->dtype; p.bits = d->bits; p.rounding = d->rounding;
    p.route = a.group < kChunk ? Route::kAnyShape
              : a.group > wide_most_elements(d->dtype) ? Route::kLarge
              : a.cpg > kMaxTeamChunks ? Route::kWide
              : a.group % kChunk != 0 ? Route::kOdd : Route::kJob;
    p.shape = p.route == Route::kOdd ? odd_team_shape_for(a.cpg, d->dtype, d->rounding, m_buf != nullptr)
                                     : team_shape_for(a.cpg);
    return p;
}

// Dequantising side: aqsgd_decode, aqsgd_grad_dequant.
struct DequantPlan {
    DequantJob job;
    int dtype;
    Route route;               // kJob, kOdd or kAnyShape
};

DequantPlan plan_dequant(const aqsgd_desc* d, int64_t batch, int64_t n_per, const uint8_t* codes,
                         const float* scales, const int64_t* ids, void* m_buf, void* out,
                         const SeenArgs& sa = SeenArgs()) {
    DequantPlan p;
    DequantJob& a = p.job;
    a.codes = codes; a.scales = scales; a.ids = ids; a.m_buf = m_buf; a.out = out; a.full = sa.full;
    a.n_per = n_per; a.gps = n_per / d->group; a.cps = n_per / kChunk;
    a.batch = static_cast<int32_t>(batch); a.group = d->group; a.cpg = d->group / kChunk; a.bits = d->bits;
    a.grid_x = a.grid_y = 1; a.rcp_grid_x = 1.0f;
    a.seen = sa.seen; a.stamp = sa.stamp;
    p.dtype = d->dtype;
    const bool odd_fits = a.group >= kChunk && odd_pieces(a, d->dtype) < kMaxOddPieces;
    p.route = a.group % kChunk == 0 ? Route::kJob : odd_fits ? Route::kOdd : Route::kAnyShape;
    return p;
}

bool smaller_than_a_wave(int shape) { return shape == kTeam8x1 || shape == kTeam16x1 || shape == kTeam32x1; }

// Steps a workgroup of a shared launch takes (`total`: steps of all its jobs; `shape`: team
// shape of the quantising ones, -1 without).  One, but for small teams (one chunk per lane) in
// large launches: a step of theirs is short next to what opens a workgroup (job lookup, sample
// id, row addresses: dependent fetches), and a launch that is several times what the chip holds
// at once (eight workgroups per compute unit, 2048) does better as one round of workgroups that
// loop, the same number of steps each, while another stream's launch runs beside it.  Measured,
// whole step in the two-stream schedule, one step -> loops: 2-bit stochastic G = 128 (6400 steps
// a launch, four each) 20.1 -> 19.1 us, 3-bit G = 64 (12288, six each) 36.8 -> 35.6.  Smaller
// launches gain more from one step each when they are alone on the chip than they lose beside
// another: 2-bit stochastic, 3200 steps, one launch a stage 27.5 -> 25.5 us, forward pair on two
// streams 13.3 -> 13.5; so the loops start at 4096.  The wider shapes (a step is four chunks per
// lane or a workgroup's row) lose from loops throughout.
int64_t steps_per_workgroup(int shape, int64_t total, int64_t launch_blocks) {
    const bool small = smaller_than_a_wave(shape);
    if (launch_blocks == 0 && small && total >= 4096) launch_blocks = 2048;
    return launch_blocks > 0 ? (total + launch_blocks - 1) / launch_blocks : 1;
}

// What a sample of a table's jobs holds of the units a workgroup's step is counted in.
int64_t whole_units(const QuantJob& a) { return a.gps; }
int64_t whole_units(const DequantJob& a) { return a.cps; }

// Workgroup numbers of a table whose jobs are all in: every job gets the grid its size
// asks for (at most max_blocks), shortened by the steps a workgroup takes (`shape`: team shape
// of the quantising jobs, -1 for one step each).  quant_step / dequant_step: units one
// workgroup step covers; units(job): those of a sample.  `threads`: lanes of a workgroup; a
// launch takes fewer than 2^32 of them along a dimension, and the jobs share one, so that
// caps each job's part.  Tells whether there is a workgroup for every step of every sample
// (else the kernel has to loop over what is left).
template <typename Units>
bool number_blocks(JobTable& t, int shape, int threads, int64_t quant_step, int64_t dequant_step, int64_t max_blocks,
                   int64_t launch_blocks, Units&& units) {
    max_blocks = std::min(max_blocks, ((int64_t{1} << 32) - 1) / threads / (t.n_quant + t.n_dequant));
    int64_t total = 0;
    auto want = [&](const auto& a, int64_t step) {
        const LaunchGeom g = geometry(units(a), step, a.batch, max_blocks);
        total += static_cast<int64_t>(g.grid_x) * g.grid_y;
    };
    for (int k = 0; k < t.n_quant; ++k) want(t.q[k], quant_step);
    for (int k = 0; k < t.n_dequant; ++k) want(t.d[k], dequant_step);
    const int64_t steps = steps_per_workgroup(shape, total, launch_blocks);
    bool covers = true;
    uint32_t blocks = 0;
    auto place = [&](auto& a, int64_t step) {
        const LaunchGeom g = geometry(units(a), step * steps, a.batch, max_blocks);
        a.grid_x = g.grid_x; a.grid_y = g.grid_y; a.rcp_grid_x = 1.0f / static_cast<float>(g.grid_x);
        covers = covers && g.grid_y == static_cast<uint32_t>(a.batch) &&
                 static_cast<int64_t>(g.grid_x) * step >= units(a);
        const uint32_t at = blocks;
        blocks += g.grid_x * g.grid_y;
        return at;
    };
    for (int k = 0; k < t.n_quant; ++k) t.q_block0[k] = place(t.q[k], quant_step);
    t.dequant_block0 = blocks;
    for (int k = 0; k < t.n_dequant; ++k) t.d_block0[k] = place(t.d[k], dequant_step);
    t.total_blocks = blocks;
    return covers;
}

// Spans of a large group: as many as give the launch about kLargeMaxBlocks workgroups, none
// shorter than one step of a workgroup.
LargeGeom large_geometry(const QuantJob& a) {
    const int64_t pieces = a.cpg;
    int64_t spans = kLargeMaxBlocks / (a.gps < kLargeMaxBlocks ? a.gps : kLargeMaxBlocks);
    spans = spans / (a.batch < spans ? a.batch : spans);
    const int64_t most = (pieces + kLargeMinSpanPieces - 1) / kLargeMinSpanPieces;
    if (spans > most) spans = most;
    LargeGeom g;
    g.span_pieces = static_cast<int32_t>(((pieces + spans - 1) / spans + kBlock - 1) / kBlock * kBlock);
    g.spans = static_cast<int32_t>((pieces + g.span_pieces - 1) / g.span_pieces);
    return g;
}

// Few wide groups with previous messages go out as spans (see split_max_kernel) where one compute
// unit's arithmetic on a group lasts longer than a second launch, up to the number of groups from
// which one workgroup each is as fast.  (Without previous messages the workgroups of one launch
// share a group: wide_share().)  One encode on the device, 8-bit, one workgroup each -> spans, in us:
//                        8 groups          32 groups         64 groups         96 groups
//   stochastic  float32   33024  12.7 ->  7.7  13.6 -> 10.2  14.5 -> 14.2  15.8 -> 17.8
//                         49152  15.2 ->  6.9  17.5 -> 10.7  19.1 -> 15.6  20.1 -> 21.9
//               bfloat16  33024  11.0 ->  7.3  11.8 ->  8.9  12.5 -> 10.6  13.1 -> 13.4
//                         65536  14.9 ->  6.7  17.8 ->  9.5  19.0 -> 13.5  21.2 -> 17.7
//   nearest     float32   33024   8.2 ->  7.2   9.9 ->  9.8  10.5 -> 13.6
//                         49152  10.5 ->  6.6  12.4 -> 10.2  14.1 -> 14.9
//               bfloat16  49152   7.4 ->  6.1   9.7 ->  8.4  10.6 -> 10.6
//                         65536   8.8 ->  6.3  11.8 ->  8.8  13.0 -> 12.4
// so 64 is the last size at which every stochastic one gains.  Nearest rounding has less to spread,
// and in a row of single calls the second launch is host time too (2.3 us): float32 stops at 32, and
// 16-bit types gain enough only in groups larger than 49152.
bool split_pays(const QuantJob& a, int dtype, int rounding) {
    const int64_t groups = a.gps * a.batch;
    if (a.m_buf == nullptr) return false;
    if (rounding == AQSGD_ROUND_STOCHASTIC) return groups <= 64;
    return groups <= 32 && (dtype == AQSGD_F32 || a.group > 49152);
}

// The same for the wide groups of a shared launch (`groups` in all, activations among them: has_buf),
// where the second launch is one for all messages and the dequantising jobs fill what the maxima leave
// idle.  A time slot of one boundary, groups of 49152, one workgroup each -> spans, in us:
//   stochastic   float16  32 groups 15.2 -> 9.4, 64 groups 17.3 -> 13.1, 96 groups 18.9 -> 16.4, 128 groups 19.5 -> 18.9
//                float32  32 groups 20.3 -> 11.7, 64 groups 22.5 -> 19.2, 96 groups 25.6 -> 24.8, 128 groups 29.2 -> 29.9
//   nearest      float32  48 groups 18.4 -> 15.1, 64 groups 19.9 -> 19.0, 96 groups 22.6 -> 24.2
//                float16   8 groups 10.8 -> 9.2, 32 groups 11.9 -> 10.5, 64 groups 13.3 -> 13.1, 96 groups 14.8 -> 15.5
//                bfloat16  8 groups 10.1 -> 9.4, 32 groups 11.1 -> 10.6, 64 groups 12.6 -> 12.9
bool split_pays_shared(int64_t groups, bool has_buf, int dtype, int rounding) {
    if (rounding == AQSGD_ROUND_STOCHASTIC) return groups <= 96;
    return has_buf && groups <= (dtype == AQSGD_F32 ? 64 : 32);
}

// Which table takes the dequantising jobs of whole groups if wide groups and a table of whole ones are to go
// out (wide forward groups, a scale for every row backward): that of the wide groups while they leave
// compute units idle, else the other.  Few wide groups that go out as spans leave little idle, too, but for
// nearest rounding of 16-bit types, whose spans are short.  A time slot of one boundary, groups of
// 49152 forward and 768 backward, with the wide ones -> with the others, in us:
//                                  32 groups      64 groups      128 groups     160 groups     256 groups
//   nearest     float16 15.3 -> 17.4  20.0 -> 20.4   26.4 -> 28.5   31.6 -> 31.3   48.6 -> 43.2
//               float32 19.4 -> 18.9  31.6 -> 29.6   43.5 -> 44.4   53.7 -> 50.7   80.3 -> 74.6
//   stochastic  bfloat16 16.0 -> 15.8  23.4 -> 20.6   30.2 -> 33.4   36.5 -> 37.2   56.8 -> 50.7
//               float32 19.6 -> 19.4  31.4 -> 29.7   44.3 -> 47.1   54.9 -> 54.3   83.0 -> 78.5
bool wide_groups_host(int64_t groups, int dtype, int rounding) {
    const bool spans = groups <= 64 && (dtype == AQSGD_F32 || rounding == AQSGD_ROUND_STOCHASTIC);
    return groups <= 144 && !spans;
}

// The rectangle of a message launched by itself: one workgroup for every sample and step if
// that stays below `cap` and the grid's second dimension, which is what this tells.
template <typename Job>
bool one_step_grid(Job& a, int64_t units, int64_t units_per_block, int64_t cap) {
    const LaunchGeom g = geometry(units, units_per_block, a.batch, cap);
    a.grid_x = g.grid_x; a.grid_y = g.grid_y;
    return g.grid_y == static_cast<uint32_t>(a.batch) && static_cast<int64_t>(g.grid_x) * units_per_block >= units;
}

// A workgroup's step is one sample's at most.  Where a sample fits one chunk per lane, the further
// chunks of a step have nothing of their own: their lanes read the row's last piece once more while
// another wave writes it, and with thousands of such workgroups in flight that is what bounds the
// launch.  So those go out with one chunk per lane.  Measured, decode at 4 bits, two chunks a lane ->
// one (as tables of one): float32 768 elements, 1024 samples 5.13 -> 4.45 us (5.62), 16384 samples
// 43.6 -> 27.8 (32.5); float16 2048 elements, 1024 samples 4.82 -> 4.71 (5.38), 16384 samples 36.6
// -> 32.1 (34.4).  With 256 samples the launch is over sooner than that matters (float32 1536
// elements 3.64 -> 3.88), and beyond one chunk per lane it costs (float32 3072 elements, 4096
// samples 26.6 -> 28.9).
bool many_short_samples(const DequantJob& a) { return a.cps <= kBlock && a.batch >= 1024; }

// Rounds of a wide group that a workgroup quantises: all of them with previous messages, which it
// updates in place; without, as few as keep the launch at one workgroup for each of the 256 compute
// units, as long as every workgroup reading a whole group costs less than the levels it saves.  One
// grad_quant, all rounds -> shared, in us: bfloat16 8 groups of 49152 4.99 -> 4.03, stochastic 6.21
// -> 4.70 (as spans in two launches 5.62), 64 groups of 40960 6.0 -> 5.3 and 9.1 -> 6.7; float16 100 groups
// of 65536 8.2 -> 8.4; float32 16 groups of 33024 5.64 -> 5.42, 70 groups of 49152 8.3 -> 9.8.
int wide_share(const QuantJob& a, int dtype, int rounding, int64_t max_blocks) {
    const int rounds = wide_rounds(dtype, a.bits, a.group);
    const int64_t groups = a.gps * a.batch, room = max_blocks < 256 ? max_blocks : 256;
    const bool pays = groups <= (dtype == AQSGD_F32 && rounding == AQSGD_ROUND_NEAREST ? 32 : 64);
    if (a.m_buf != nullptr || !pays || room < 2 * groups) return rounds;
    const int64_t parts = room / groups;
    return static_cast<int>((rounds + parts - 1) / parts);
}

// A quantising message outside the job kernels' range.
hipError_t launch_quant_alone(QuantPlan& p, int64_t max_blocks, int64_t launch_blocks, hipStream_t stream) {
    QuantJob& a = p.job;
    LaunchGeom g;
    switch (p.route) {
    case Route::kOdd: {
        const int64_t cap = launch_blocks > 0 && launch_blocks < max_blocks ? launch_blocks : max_blocks;
        const bool covers = one_step_grid(a, a.gps, groups_per_block_step(p.shape), cap);
        return launch_quant_single(p.dtype, p.rounding, p.shape, covers, false, a, stream);
    }
    case Route::kWide:
        if (split_pays(a, p.dtype, p.rounding)) {
            const LargeGeom sg = split_geometry(a);
            if (one_step_grid(a, a.gps * sg.spans, 1, max_blocks))
                return launch_quant_split(p.dtype, p.rounding, a, sg, stream);
        }
        if (one_step_grid(a, a.gps, 1, max_blocks)) {
            const int rounds = wide_rounds(p.dtype, a.bits, a.group);
            const int share = wide_share(a, p.dtype, p.rounding, max_blocks);
            return launch_quant_wide(p.dtype, p.rounding, (rounds + share - 1) / share, share, a, stream);
        }
        [[fallthrough]];                                 // too many for a grid: the kernels that loop
    case Route::kLarge: {
        const LargeGeom lg = large_geometry(a);
        g = geometry(a.gps * lg.spans, 1, a.batch, max_blocks);
        a.grid_x = g.grid_x; a.grid_y = g.grid_y;
        return launch_quant_large(p.dtype, p.rounding, a, lg, stream);
    }
    default:
        g = geometry(a.gps, kBlock, a.batch, max_blocks);
        a.grid_x = g.grid_x; a.grid_y = g.grid_y;
        return launch_quant_anyshape(p.dtype, p.bits, p.rounding, a, stream);
    }
}

// Gradients of odd float32 groups in whole pieces, alone (all others stream): time streaming over time through,
// the same output every time, 33 MB written 0.98, 65 MB 1.06, 98 MB 1.11 (the last-level cache holds such an
// output), other outputs 1.00 to 1.01.  With previous messages 0.99 to 1.01.
constexpr int64_t kThroughOddBytes = int64_t{48} << 20;

bool odd_writes_through(const DequantJob& a, int dtype) {
    return dtype == AQSGD_F32 && a.m_buf == nullptr && a.group % kUnit == 0 && a.batch * a.n_per * 4 >= kThroughOddBytes;
}

hipError_t launch_dequant_alone(DequantPlan& p, int64_t max_blocks, hipStream_t stream) {
    DequantJob& a = p.job;
    if (p.route == Route::kOdd) {
        const bool covers = one_step_grid(a, odd_pieces(a, p.dtype), static_cast<int64_t>(kBlock) * kOddUnroll, max_blocks);
        return launch_dequant_odd(p.dtype, covers, covers && odd_writes_through(a, p.dtype), a, stream);
    }
    const LaunchGeom g = geometry(a.gps, kBlock, a.batch, max_blocks);
    a.grid_x = g.grid_x; a.grid_y = g.grid_y;
    return launch_dequant_anyshape(p.dtype, a, stream);
}

// Which launches write previous messages and reconstructions through the L2 (see store16): those whose
// rows (and groups, on the quantising side, where a team of lanes stores its own) are whole 128-byte
// lines and that write more than about the eight L2s hold in lines that have not left yet.
//
// Shared launches, a time slot on one stream, through -> streaming: bfloat16 [18,175,128], four boundaries,
// 15 MB written 10.3 -> 9.1 us; [1,1537,384], two boundaries, 11 MB 7.2 -> 6.5; of whole lines, 60 MB and more,
// equal within 2 % and better through with another stream beside it.  One job that is not of whole lines
// makes the table stream: float32 [1,2048,2704] G = 2704 (groups of 84 and a half lines, whole
// rows), four boundaries, 142 -> 125 (only its encode streaming 125); [8,512,2048] G = 16 79 -> 66 (75); float16
// [8,512,2048] G = 32 31.8 -> 30.8 (31.3).
constexpr int64_t kThroughBytes = int64_t{24} << 20;

int64_t bytes_written(const QuantJob& a, int64_t eb) {
    return a.batch * a.n_per * (a.m_buf ? 8 * eb + a.bits : a.bits) / 8;
}
int64_t bytes_written(const DequantJob& a, int64_t eb) { return a.batch * a.n_per * eb * (a.m_buf ? 2 : 1); }
constexpr int64_t kLineBytes = 128;
bool whole_lines(const QuantJob& a, int64_t eb) {
    return a.n_per * eb % kLineBytes == 0 && a.group * eb % kLineBytes == 0;
}
bool whole_lines(const DequantJob& a, int64_t eb) { return a.n_per * eb % kLineBytes == 0; }

// A reconstruction alone.  Large ones (measured in a row of four calls, through -> streaming: float32
// [8,2048,4096] 362 -> 366 us, bfloat16 [32,256,1536] 46.3 -> 46.8, first visits of float16 [4,1024,1600], 26 MB
// written, 17.4 -> 17.7), and gradients of the sizes of which much streams out of the L2s before the launch
// ends when the output is the same buffer every time.  Time of a grad_dequant streaming over time through, by the MiB
// written (G = 64 to 4096, geometric means over four and, of 16 bits, eight):
//                               8     10     12     14     16     18     20     22
//   16 bits  same output      0.95   0.94   1.05   1.06   1.01   0.97   0.97   0.94
//            others           0.94   0.93   0.95   0.96   0.97   0.97   0.98   0.98
//   float32  same output      0.95   0.94   1.15   1.10   1.11   1.05   1.00   1.00
//            others           0.95   0.95   0.95   0.96   0.96   0.98   0.98   1.00
// A decode, which writes m and out, has no such sizes (0.97 to 1.02 from 12 MiB written on).
constexpr int64_t kThroughGradBytes = int64_t{11} << 20;
constexpr int64_t stream_grad_bytes(int dtype) { return int64_t{dtype == AQSGD_F32 ? 19 : 17} << 20; }

bool writes_through(const DequantJob& a, int dtype) {
    const int64_t eb = dtype == AQSGD_F32 ? 4 : 2, bytes = bytes_written(a, eb);
    const bool grad = a.m_buf == nullptr && bytes >= kThroughGradBytes && bytes < stream_grad_bytes(dtype);
    return (bytes >= kThroughBytes || grad) && whole_lines(a, eb);
}

// An encode alone: time streaming over time through, by the MiB of m it writes (4 bits, G = 64 to 4096, both
// roundings, geometric means over seven to twenty of them; the same rows every time, which the last-level
// cache keeps, and others every time, which it does not):
//                          2      8-10     12-14     16-18      22      28-40
//   16 bits  same rows   0.89   0.92-0.94 0.95-0.97 1.02-1.03  1.05   1.03-1.04
//            others      0.99   0.98-1.00   1.00    0.99-1.00  1.00     1.02
//   float32  same rows   0.88   0.79-0.80 0.79-0.87 0.95-0.97  1.00     1.02
//            others      0.97     1.00    0.99-1.00   0.99     0.99   1.00-1.01
// and beyond, m of 67 MB and more, others 1.01 to 1.02 (one float32 [8,2048,4096] 125.9 us through, 127.7
// streaming, float16 [16,2048,2048] 64.3 and 65.5).  The lines lie at 16 and 22 MiB of m.  3 bits the same:
// bfloat16 [8,1024,2048] G = 256, 1.02 and 1.01, stochastic 1.07 and 1.02.  Groups that are no octets stream.
constexpr int64_t through_encode_bytes(int dtype) { return int64_t{dtype == AQSGD_F32 ? 24 : 20} << 20; }

bool writes_through(const QuantJob& a, int dtype) {
    const int64_t eb = dtype == AQSGD_F32 ? 4 : 2;
    return a.m_buf && bytes_written(a, eb) >= through_encode_bytes(dtype) && whole_lines(a, eb);
}

// A table's jobs are stored alike: through if all that hold such stores are of whole lines.
bool writes_through(const JobTable& t, int dtype) {
    const int64_t eb = dtype == AQSGD_F32 ? 4 : 2;
    int64_t bytes = 0;
    bool lines = true;
    for (int k = 0; k < t.n_quant; ++k) {
        bytes += bytes_written(t.q[k], eb);
        lines = lines && (t.q[k].m_buf == nullptr || whole_lines(t.q[k], eb));
    }
    for (int k = 0; k < t.n_dequant; ++k) {
        bytes += bytes_written(t.d[k], eb);
        lines = lines && whole_lines(t.d[k], eb);
    }
    return lines && bytes >= kThroughBytes;
}

// A message that comes alone.  Without lists: a small message's call is over on the device in 2 to 3 us,
// and the host's share of a call is what a row of them waits for.  The single-message kernels open
// sooner (see aqsgd_single.h); their workgroups do one step each, so a message that would pass the
// caps on a grid, or one in a sweep of launch sizes, goes out as a table of one instead (`false`).
bool launch_alone(QuantPlan& q, int64_t max_blocks, int64_t launch_blocks, hipStream_t stream, hipError_t& err) {
    if (q.route != Route::kJob) {
        err = launch_quant_alone(q, max_blocks, launch_blocks, stream);
        return true;
    }
    if (launch_blocks != 0 || !one_step_grid(q.job, q.job.gps, groups_per_block_step(q.shape), max_blocks)) return false;
    err = launch_quant_single(q.dtype, q.rounding, q.shape, true, writes_through(q.job, q.dtype), q.job, stream);
    return true;
}

bool launch_alone(DequantPlan& d, int64_t max_blocks, int64_t launch_blocks, hipStream_t stream, hipError_t& err) {
    if (d.route != Route::kJob) {
        err = launch_dequant_alone(d, max_blocks, stream);
        return true;
    }
    const int chunks = many_short_samples(d.job) ? 1 : dequant_unroll_knob().load(std::memory_order_relaxed);
    if (launch_blocks != 0 || !one_step_grid(d.job, d.job.cps, static_cast<int64_t>(kBlock) * chunks, max_blocks)) return false;
    err = launch_dequant_single(d.dtype, chunks, writes_through(d.job, d.dtype), d.job, stream);
    return true;
}

// A job's workgroup numbers must be exact in binary32 (place_in_job).
int64_t blocks_cap() {
    const int64_t knob = max_blocks_knob().load(std::memory_order_relaxed);
    return knob < (int64_t{1} << 24) ? knob : (int64_t{1} << 24) - 1;
}

// The launches of a set of independent messages: quantising jobs that share dtype,
// rounding mode and team shape go into one grid, together with the dequantising
// jobs of that dtype that are still waiting; odd and wide groups likewise among themselves;
// dequantising jobs without such a host get a grid of their own; what is left (groups of 1 to 7
// elements, those beyond a workgroup, odd reconstructions without a host) is launched one by one.
int launch_plans(std::vector<QuantPlan>& qs, std::vector<DequantPlan>& ds, hipStream_t stream) {
    const int64_t max_blocks = blocks_cap();
    const int unroll = dequant_unroll_knob().load(std::memory_order_relaxed);
    std::vector<bool> q_done(qs.size(), false), d_done(ds.size(), false);
    hipError_t err = hipSuccess;

    const int64_t launch_blocks = launch_blocks_knob().load(std::memory_order_relaxed);
    if (qs.size() + ds.size() == 1 &&
        (qs.empty() ? launch_alone(ds[0], max_blocks, launch_blocks, stream, err)
                    : launch_alone(qs[0], max_blocks, launch_blocks, stream, err)))
        return err == hipSuccess ? AQSGD_OK : AQSGD_ERR_LAUNCH;
    const auto whole = [](const auto& a) { return whole_units(a); };
    auto add_dequant = [&](JobTable& t, int dtype, Route route, size_t* taken = nullptr) {
        for (size_t k = 0; k < ds.size() && t.n_dequant < kMaxDequantJobs; ++k) {
            if (d_done[k] || ds[k].route != route || ds[k].dtype != dtype) continue;
            if (taken) taken[t.n_dequant] = k;
            t.d[t.n_dequant++] = ds[k].job;
            d_done[k] = true;
        }
    };
    // Odd and wide groups: those of one kind (dtype, rounding mode; odd ones also team shape) and
    // the dequantising jobs that are ready with them as one table, if that has more than one
    // job and a workgroup for each of their steps.
    auto launch_shared = [&](size_t i) {
        const QuantPlan& lead = qs[i];
        const bool odd = lead.route == Route::kOdd;
        if ((!odd && lead.route != Route::kWide) || launch_blocks > 0) return false;
        JobTable t;
        t.n_quant = t.n_dequant = 0;
        size_t taken_q[kMaxQuantJobs], taken_d[kMaxDequantJobs];     // no list: something may be enqueued by now
        int64_t groups = 0;
        bool has_buf = false;
        for (size_t k = i; k < qs.size() && t.n_quant < kMaxQuantJobs; ++k) {
            const QuantPlan& c = qs[k];
            if (q_done[k] || c.route != lead.route || c.dtype != lead.dtype || c.rounding != lead.rounding ||
                (odd && c.shape != lead.shape))
                continue;
            groups += c.job.gps * c.job.batch;
            has_buf = has_buf || c.job.m_buf != nullptr;
            taken_q[t.n_quant] = k;
            t.q[t.n_quant++] = c.job;
            q_done[k] = true;
        }
        bool waiting = false;                            // a table of whole groups is still to come
        for (size_t k = i; k < qs.size(); ++k)
            waiting = waiting || (!q_done[k] && qs[k].route == Route::kJob && qs[k].dtype == lead.dtype);
        if (odd || !waiting || wide_groups_host(groups, lead.dtype, lead.rounding))
            add_dequant(t, lead.dtype, odd ? Route::kOdd : Route::kJob, taken_d);
        bool covers = t.n_quant + t.n_dequant > 1;
        if (covers && odd) {
            struct {
                int dtype;
                int64_t operator()(const QuantJob& a) const { return a.gps; }
                int64_t operator()(const DequantJob& a) const { return odd_pieces(a, dtype); }
            } units{lead.dtype};
            covers = number_blocks(t, -1, threads_of_shape(lead.shape), groups_per_block_step(lead.shape),
                                   static_cast<int64_t>(threads_of_shape(lead.shape)) * kOddUnroll, max_blocks, 0, units);
            if (covers) err = launch_odd_jobs(lead.dtype, lead.rounding, lead.shape, t, stream);
        } else if (covers && split_pays_shared(groups, has_buf, lead.dtype, lead.rounding)) {
            struct {
                int64_t operator()(const QuantJob& a) const { return a.gps * split_geometry(a).spans; }
                int64_t operator()(const DequantJob& a) const { return a.cps; }
            } units;
            covers = number_blocks(t, -1, kBlock, 1, static_cast<int64_t>(kBlock) * kHostedDequantUnroll, max_blocks, 0, units);
            if (covers) err = launch_split_jobs(lead.dtype, lead.rounding, t, stream);
        } else if (covers) {
            covers = number_blocks(t, -1, kWideThreads, 1, static_cast<int64_t>(kWideThreads) * kHostedDequantUnroll, max_blocks, 0,
                                   whole);
            if (covers) err = launch_wide_jobs(lead.dtype, lead.rounding, t, stream);
        }
        if (!covers) {
            for (int k = 0; k < t.n_quant; ++k) q_done[taken_q[k]] = false;
            for (int k = 0; k < t.n_dequant; ++k) d_done[taken_d[k]] = false;
        }
        return covers;
    };

    for (size_t i = 0; i < qs.size() && err == hipSuccess; ++i) {
        if (q_done[i]) continue;
        QuantPlan& lead = qs[i];
        if (lead.route != Route::kJob) {
            if (launch_shared(i)) continue;
            err = launch_quant_alone(lead, max_blocks, launch_blocks, stream);
            q_done[i] = true;
            continue;
        }
        JobTable t;
        t.n_quant = t.n_dequant = 0;
        bool three = false;                              // a 3-bit job among them
        for (size_t k = i; k < qs.size() && t.n_quant < kMaxQuantJobs; ++k) {
            const QuantPlan& c = qs[k];
            if (q_done[k] || c.route != Route::kJob || c.shape != lead.shape || c.dtype != lead.dtype ||
                c.rounding != lead.rounding)
                continue;
            three = three || c.bits == 3;
            t.q[t.n_quant++] = c.job;
            q_done[k] = true;
        }
        add_dequant(t, lead.dtype, Route::kJob);
        const bool covers = number_blocks(t, lead.shape, threads_of_shape(lead.shape), groups_per_block_step(lead.shape),
                                          static_cast<int64_t>(threads_of_shape(lead.shape)) * kHostedDequantUnroll,
                                          max_blocks, launch_blocks, whole);
        const TableKind kind = covers ? (three ? kTableOneStepThree : kTableOneStep)
                                      : (three ? kTableLoopsThree : kTableLoops);
        const bool through = (covers || smaller_than_a_wave(lead.shape)) && writes_through(t, lead.dtype);
        err = launch_codec_jobs(lead.dtype, lead.rounding, lead.shape, kind, through, t, stream);
    }
    for (size_t i = 0; i < ds.size() && err == hipSuccess; ++i) {
        if (d_done[i]) continue;
        if (ds[i].route != Route::kJob) {
            err = launch_dequant_alone(ds[i], max_blocks, stream);
            d_done[i] = true;
            continue;
        }
        JobTable t;
        t.n_quant = t.n_dequant = 0;
        add_dequant(t, ds[i].dtype, Route::kJob);
        number_blocks(t, -1, kBlock, 1, static_cast<int64_t>(kBlock) * unroll, max_blocks, launch_blocks, whole);
        err = launch_dequant_jobs(ds[i].dtype, unroll, writes_through(t, ds[i].dtype), t, stream);
    }
    return err == hipSuccess ? AQSGD_OK : AQSGD_ERR_LAUNCH;
}

// No C++ exception leaves a C entry: a caller in another language cannot catch it, and one that
// has let go of a lock (an interpreter's) could not take it up again.  What can be thrown is the
// want of host memory for the lists of messages, before anything is enqueued.
template <typename F>
int without_exceptions(F&& f) {
    try {
        return f();
    } catch (...) {
        return AQSGD_ERR_LAUNCH;
    }
}

template <typename Plan>
int launch_one(Plan p, hipStream_t stream) {
    hipError_t err = hipSuccess;
    if (launch_alone(p, blocks_cap(), launch_blocks_knob().load(std::memory_order_relaxed), stream, err))
        return err == hipSuccess ? AQSGD_OK : AQSGD_ERR_LAUNCH;
    return without_exceptions([&] {
        std::vector<QuantPlan> qs;
        std::vector<DequantPlan> ds;
        if constexpr (std::is_same_v<Plan, QuantPlan>) qs.push_back(p);
        else ds.push_back(p);
        return launch_plans(qs, ds, stream);
    });
}

// Row copy for the uncompressed first visit of aqsgd_seed: m_buf[ids[i]] <- act[i].
// V = 16 bytes per lane and step (streaming accesses) when the row size allows it,
// else one element.
template <typename V>
__global__ __launch_bounds__(kBlock)
void seed_rows_kernel(const V* act, const int64_t* ids, V* m_buf, int64_t units_per_row, int batch) {
    for (int i = blockIdx.y; i < batch; i += gridDim.y) {
        const int64_t row = sample_id(ids, i);
        const V* src = act + static_cast<int64_t>(i) * units_per_row;
        V* dst = m_buf + row * units_per_row;
        for (int64_t c = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; c < units_per_row;
             c += static_cast<int64_t>(gridDim.x) * kBlock) {
            if constexpr (sizeof(V) == 16) {
                const V v = __builtin_nontemporal_load(src + c);
                // written through at every size: streaming, in us, float16 [4,32768] 2.07 -> 2.18, [4,1638400] 3.45 -> 3.82,
                // bfloat16 [32,393216] 5.4 -> 8.9 (the same rows every time; others 10.15 -> 10.09), float32 [8,8388608] 81.6 -> 80.3
                store16(dst + c, v, true);
            } else {
                dst[c] = src[c];
            }
        }
    }
}

template <typename V>
hipError_t launch_seed_rows_as(const aqsgd_desc* d, int64_t row_bytes, const void* act, const int64_t* ids,
                               void* m_buf, hipStream_t s) {
    const int64_t units = row_bytes / static_cast<int64_t>(sizeof(V));
    const LaunchGeom g = geometry(units, static_cast<int64_t>(kBlock) * (sizeof(V) == 16 ? 2 : 4), d->batch,
                            max_blocks_knob().load(std::memory_order_relaxed));
    return launch_kernel(seed_rows_kernel<V>, dim3(g.grid_x, g.grid_y), dim3(kBlock), s,
                         static_cast<const V*>(act), ids, static_cast<V*>(m_buf), units,
                         static_cast<int>(d->batch));
}

hipError_t launch_seed_rows(const aqsgd_desc* d, const void* act, const int64_t* ids, void* m_buf,
                            hipStream_t s) {
    const int64_t eb = d->dtype == AQSGD_F32 ? 4 : 2;
    const int64_t row_bytes = d->n_per * eb;
    if (row_bytes % 16 == 0) return launch_seed_rows_as<u32x4_t>(d, row_bytes, act, ids, m_buf, s);
    if (eb == 4) return launch_seed_rows_as<uint32_t>(d, row_bytes, act, ids, m_buf, s);
    return launch_seed_rows_as<uint16_t>(d, row_bytes, act, ids, m_buf, s);
}

int check_encode(const aqsgd_desc* d, const void* act, const int64_t* ids, const void* m_buf,
                 const uint8_t* codes, const float* scales) {
    const int rc = check_desc(d, true);
    if (rc != AQSGD_OK || d->batch == 0) return rc;
    if (!act || !ids || !m_buf || !codes || !scales) return AQSGD_ERR_NULL;
    if (!aligned(act, 16) || !aligned(m_buf, 16) || !aligned(codes, 16) || !aligned(scales, 4) ||
        !aligned(ids, 8))
        return AQSGD_ERR_ALIGN;
    return AQSGD_OK;
}

int check_decode(const aqsgd_desc* d, const uint8_t* codes, const float* scales, const int64_t* ids,
                 const void* m_buf, const void* out) {
    const int rc = check_desc(d, true);
    if (rc != AQSGD_OK || d->batch == 0) return rc;
    if (!codes || !scales || !ids || !m_buf || !out) return AQSGD_ERR_NULL;
    if (!aligned(out, 16) || !aligned(m_buf, 16) || !aligned(codes, 16) || !aligned(scales, 4) ||
        !aligned(ids, 8))
        return AQSGD_ERR_ALIGN;
    return AQSGD_OK;
}

int check_grad_quant(const aqsgd_desc* d, const void* grad, const uint8_t* codes, const float* scales) {
    const int rc = check_desc(d, false);
    if (rc != AQSGD_OK || d->batch == 0) return rc;
    if (!grad || !codes || !scales) return AQSGD_ERR_NULL;
    if (!aligned(grad, 16) || !aligned(codes, 16) || !aligned(scales, 4)) return AQSGD_ERR_ALIGN;
    return AQSGD_OK;
}

int check_grad_dequant(const aqsgd_desc* d, const uint8_t* codes, const float* scales, const void* out) {
    const int rc = check_desc(d, false);
    if (rc != AQSGD_OK || d->batch == 0) return rc;
    if (!codes || !scales || !out) return AQSGD_ERR_NULL;
    if (!aligned(out, 16) || !aligned(codes, 16) || !aligned(scales, 4)) return AQSGD_ERR_ALIGN;
    return AQSGD_OK;
}

// The backward message has no per-sample rows to gather, and n_per is a multiple of
// the group, so the call tensor is treated as one long sample.
QuantPlan plan_grad_quant(const aqsgd_desc* d, const void* grad, uint8_t* codes, float* scales) {
    const int64_t n = d->batch * d->n_per;
    const bool flat = n <= (int64_t{1} << 34);
    return plan_quant(d, flat ? 1 : d->batch, flat ? n : d->n_per, grad, nullptr, nullptr, codes, scales);
}

DequantPlan plan_grad_dequant(const aqsgd_desc* d, const uint8_t* codes, const float* scales, void* out) {
    const int64_t n = d->batch * d->n_per;
    const bool flat = n <= (int64_t{1} << 34);
    return plan_dequant(d, flat ? 1 : d->batch, flat ? n : d->n_per, codes, scales, nullptr, nullptr, out);
}

int lowbit_shape_for(int cpg) {
    if (cpg <= 8) return kLb8x1;
    if (cpg <= 16) return kLb16x1;
    if (cpg <= 32) return kLb32x1;
    if (cpg <= 64) return kLb64x1;
    if (cpg <= 128) return kLb64x2;
    if (cpg <= 192) return kLb64x3;
    if (cpg <= 256) return kLb64x4;
    if (cpg <= 512) return kLb256x2;
    if (cpg <= 1024) return kLb256x4;
    return kLb1024x2;
}

int lowbit_teams_per_block(int shape) {
    switch (shape) {
    case kLb8x1: return kBlock / 8;
    case kLb16x1: return kBlock / 16;
    case kLb32x1: return kBlock / 32;
    case kLb64x1: case kLb64x2: case kLb64x3: case kLb64x4: return kBlock / 64;
    default: return 1;
    }
}

int check_lowbit(const aqsgd_desc* d, int32_t m_bits) {
    const int rc = check_desc(d, true);
    if (rc != AQSGD_OK) return rc;
    if (m_bits != 2 && m_bits != 8) return AQSGD_ERR_BITS;
    if (d->group % kChunk != 0 || d->group / kChunk > kMaxLowbitChunks) return AQSGD_ERR_GROUP;
    return AQSGD_OK;
}

// A low-precision receiver's reconstruction, 16-bit types of whole 128-byte lines: time streaming over time
// through, by the MiB written (float16 and bfloat16, G = 64 to 1024, m at 8 and 2 bits; the same rows every
// time, and others every time; medians of twelve):
//                 1      2      4      6      10     16     32
//   same rows    0.98   1.02   1.06   1.06   1.05   1.04   1.02
//   others       0.97   1.00   1.03   1.03   1.02   1.02   1.01
// (rows of 1600, 3.2 MB, 0.97.)  The kernel is bound by arithmetic, so what streams waits for the end.  Rows or
// groups that are no whole lines stream: bfloat16 [7,1001,2008] 14.2 us through, 9.8 streaming.
constexpr int64_t kThroughLowbitBytes = int64_t{4} << 20;

bool lowbit_writes_through(const LowbitArgs& a, int dtype) {
    return dtype != AQSGD_F32 && a.batch * a.n_per * 2 >= kThroughLowbitBytes && a.n_per * 2 % kLineBytes == 0 &&
           a.group * 2 % kLineBytes == 0;
}

int run_lowbit(const aqsgd_desc* d, int32_t m_bits, bool sender, const void* act, void* out,
               const int64_t* ids, uint8_t* m_codes, float* m_scales, uint8_t* codes, float* scales,
               hipStream_t stream) {
    LowbitArgs a;
    a.act = act; a.out = out; a.ids = ids; a.m_codes = m_codes; a.m_scales = m_scales;
    a.codes = codes; a.scales = scales;
    a.n_per = d->n_per; a.gps = d->n_per / d->group;
    a.batch = static_cast<int32_t>(d->batch); a.group = d->group; a.cpg = d->group / kChunk;
    a.stochastic = d->rounding == AQSGD_ROUND_STOCHASTIC; a.seed = d->rng_seed;
    a.through = !sender && lowbit_writes_through(a, d->dtype);
    const int shape = lowbit_shape_for(a.cpg);
    const hipError_t err = launch_lowbit(d->dtype, d->bits, m_bits, shape, sender,
                                         geometry(a.gps, lowbit_teams_per_block(shape), d->batch,
                                                  max_blocks_knob().load(std::memory_order_relaxed)),
                                         a, stream);
    return err == hipSuccess ? AQSGD_OK : AQSGD_ERR_LAUNCH;
}

int check_topk(const aqsgd_desc* d, int32_t keep) {
    const int rc = check_desc(d, false);
    if (rc != AQSGD_OK) return rc;
    if (d->bits != kTopkBits) return AQSGD_ERR_BITS;
    if (d->group % kChunk != 0 || d->group > kTopkMaxGroup) return AQSGD_ERR_GROUP;
    if (keep < 1 || keep > d->group) return AQSGD_ERR_SHAPE;
    return AQSGD_OK;
}

int run_topk(const aqsgd_desc* d, int32_t keep, bool sender, const void* grad, void* out, uint8_t* bitmap,
             uint8_t* codes, float* scales, hipStream_t stream) {
    TopkArgs a;
    a.grad = grad; a.out = out; a.bitmap = bitmap; a.codes = codes; a.scales = scales;
    a.n_groups = d->batch * (d->n_per / d->group);
    a.group = d->group; a.cpg = d->group / kChunk; a.keep = keep;
    a.stochastic = d->rounding == AQSGD_ROUND_STOCHASTIC; a.seed = d->rng_seed;
    const TopkSmallShape small = topk_small_shape(d->dtype, sender, a.cpg, a.n_groups);
    if (small.lanes > 0) {
        const LaunchGeom g = geometry(a.n_groups, kWave / small.lanes, 1,
                                      max_blocks_knob().load(std::memory_order_relaxed));
        const hipError_t err = launch_topk_small(d->dtype, small, sender, g.grid_x, a, stream);
        return err == hipSuccess ? AQSGD_OK : AQSGD_ERR_LAUNCH;
    }
    const int cpl = a.cpg <= kWave ? 1 : (a.cpg <= 2 * kWave ? 2 : (a.cpg <= 3 * kWave ? 3 : 4));
    const LaunchGeom g = geometry(a.n_groups, kTopkBlock / kWave, 1,
                                  max_blocks_knob().load(std::memory_order_relaxed));
    const hipError_t err = launch_topk(d->dtype, cpl, sender, g.grid_x, a, stream);
    return err == hipSuccess ? AQSGD_OK : AQSGD_ERR_LAUNCH;
}

// Every job is checked before anything is enqueued.
int run_jobs(const aqsgd_job* jobs, int32_t n_jobs, hipStream_t stream) {
    std::vector<QuantPlan> qs;
    std::vector<DequantPlan> ds;
    for (int32_t k = 0; k < n_jobs; ++k) {
        const aqsgd_job& j = jobs[k];
        const aqsgd_desc* d = &j.desc;
        int rc;
        switch (j.kind) {
        case AQSGD_JOB_ENCODE:
            rc = check_encode(d, j.src, j.sample_ids, j.m_buf, j.codes, j.scales);
            if (rc == AQSGD_OK && d->batch > 0)
                qs.push_back(plan_quant(d, d->batch, d->n_per, j.src, j.sample_ids, j.m_buf, j.codes, j.scales));
            break;
        case AQSGD_JOB_DECODE:
            rc = check_decode(d, j.codes, j.scales, j.sample_ids, j.m_buf, j.out);
            if (rc == AQSGD_OK && d->batch > 0)
                ds.push_back(plan_dequant(d, d->batch, d->n_per, j.codes, j.scales, j.sample_ids, j.m_buf, j.out));
            break;
        case AQSGD_JOB_GRAD_QUANT:
            rc = check_grad_quant(d, j.src, j.codes, j.scales);
            if (rc == AQSGD_OK && d->batch > 0) qs.push_back(plan_grad_quant(d, j.src, j.codes, j.scales));
            break;
        case AQSGD_JOB_GRAD_DEQUANT:
            rc = check_grad_dequant(d, j.codes, j.scales, j.out);
            if (rc == AQSGD_OK && d->batch > 0) ds.push_back(plan_grad_dequant(d, j.codes, j.scales, j.out));
            break;
        case AQSGD_JOB_ENCODE_SEEN: {
            rc = check_encode(d, j.src, j.sample_ids, j.m_buf, j.codes, j.scales);
            if (rc == AQSGD_OK && j.stamp == 0) rc = AQSGD_ERR_SHAPE;
            if (rc != AQSGD_OK || d->batch == 0) break;
            if (!j.seen || !j.first) { rc = AQSGD_ERR_NULL; break; }
            if (!aligned(j.first, 4) || !aligned(j.seen, 4)) { rc = AQSGD_ERR_ALIGN; break; }
            SeenArgs sa;
            sa.seen = j.seen; sa.first = j.first; sa.stamp = j.stamp;
            qs.push_back(plan_quant(d, d->batch, d->n_per, j.src, j.sample_ids, j.m_buf, j.codes, j.scales, sa));
            break;
        }
        case AQSGD_JOB_DECODE_SEEN: {
            rc = check_decode(d, j.codes, j.scales, j.sample_ids, j.m_buf, j.out);
            if (rc == AQSGD_OK && j.stamp == 0) rc = AQSGD_ERR_SHAPE;
            if (rc != AQSGD_OK || d->batch == 0) break;
            if (!j.seen || !j.full) { rc = AQSGD_ERR_NULL; break; }
            if (!aligned(j.full, 16) || !aligned(j.seen, 4)) { rc = AQSGD_ERR_ALIGN; break; }
            SeenArgs sa;
            sa.seen = j.seen; sa.full = j.full; sa.stamp = j.stamp;
            ds.push_back(plan_dequant(d, d->batch, d->n_per, j.codes, j.scales, j.sample_ids, j.m_buf, j.out, sa));
            break;
        }
        default:
            rc = AQSGD_ERR_SHAPE;
        }
        if (rc != AQSGD_OK) return rc;
    }
    return launch_plans(qs, ds, stream);
}

__global__ void check_ids_kernel(const int64_t* ids, int64_t batch, int64_t n_samples, int32_t* flag) {
    int bad = 0;
    for (int64_t i = threadIdx.x + static_cast<int64_t>(blockIdx.x) * blockDim.x; i < batch;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t v = ids[i];
        if (v < 0 || v >= n_samples) bad |= 1;
        for (int64_t j = 0; j < i; ++j)
            if (ids[j] == v) bad |= 2;
    }
    if (bad) atomicOr(flag, bad);
}

}  // namespace
}  // namespace aqsgd

using namespace aqsgd;

extern "C" {

size_t aqsgd_codes_bytes(const aqsgd_desc* d) {
    if (check_desc(d, false) != AQSGD_OK) return 0;
    return static_cast<size_t>(d->batch) * static_cast<size_t>(d->n_per) * d->bits / 8;
}

size_t aqsgd_scales_count(const aqsgd_desc* d) {
    if (check_desc(d, false) != AQSGD_OK) return 0;
    return static_cast<size_t>(d->batch) * static_cast<size_t>(d->n_per / d->group);
}

int aqsgd_encode(const aqsgd_desc* d, const void* act, const int64_t* sample_ids, void* m_buf,
                 uint8_t* codes, float* scales, void* stream) {
    const int rc = check_encode(d, act, sample_ids, m_buf, codes, scales);
    if (rc != AQSGD_OK || d->batch == 0) return rc;
    return launch_one(plan_quant(d, d->batch, d->n_per, act, sample_ids, m_buf, codes, scales),
                      static_cast<hipStream_t>(stream));
}

int aqsgd_decode(const aqsgd_desc* d, const uint8_t* codes, const float* scales,
                 const int64_t* sample_ids, void* m_buf, void* out, void* stream) {
    const int rc = check_decode(d, codes, scales, sample_ids, m_buf, out);
    if (rc != AQSGD_OK || d->batch == 0) return rc;
    return launch_one(plan_dequant(d, d->batch, d->n_per, codes, scales, sample_ids, m_buf, out),
                      static_cast<hipStream_t>(stream));
}

int aqsgd_grad_quant(const aqsgd_desc* d, const void* grad, uint8_t* codes, float* scales,
                     void* stream) {
    const int rc = check_grad_quant(d, grad, codes, scales);
    if (rc != AQSGD_OK || d->batch == 0) return rc;
    return launch_one(plan_grad_quant(d, grad, codes, scales), static_cast<hipStream_t>(stream));
}

int aqsgd_grad_dequant(const aqsgd_desc* d, const uint8_t* codes, const float* scales, void* out,
                       void* stream) {
    const int rc = check_grad_dequant(d, codes, scales, out);
    if (rc != AQSGD_OK || d->batch == 0) return rc;
    return launch_one(plan_grad_dequant(d, codes, scales, out), static_cast<hipStream_t>(stream));
}

int aqsgd_run_jobs(const aqsgd_job* jobs, int32_t n_jobs, void* stream) {
    if (n_jobs < 0) return AQSGD_ERR_SHAPE;
    if (n_jobs == 0) return AQSGD_OK;
    if (!jobs) return AQSGD_ERR_NULL;
    return without_exceptions([&] { return run_jobs(jobs, n_jobs, static_cast<hipStream_t>(stream)); });
}

int aqsgd_seed(const aqsgd_desc* d, const void* act, const int64_t* sample_ids, void* m_buf,
               void* stream) {
    const int rc = check_desc(d, true);
    if (rc != AQSGD_OK) return rc;
    if (d->batch == 0) return AQSGD_OK;
    if (!act || !sample_ids || !m_buf) return AQSGD_ERR_NULL;
    if (!aligned(act, 16) || !aligned(m_buf, 16) || !aligned(sample_ids, 8)) return AQSGD_ERR_ALIGN;
    const hipError_t err = launch_seed_rows(d, act, sample_ids, m_buf, static_cast<hipStream_t>(stream));
    return err == hipSuccess ? AQSGD_OK : AQSGD_ERR_LAUNCH;
}

int aqsgd_encode_seen(const aqsgd_desc* d, const void* act, const int64_t* sample_ids, void* m_buf,
                      uint32_t* seen, uint32_t stamp, int32_t* first, uint8_t* codes, float* scales,
                      void* stream) {
    const int rc = check_encode(d, act, sample_ids, m_buf, codes, scales);
    if (rc != AQSGD_OK) return rc;
    if (stamp == 0) return AQSGD_ERR_SHAPE;
    if (d->batch == 0) return AQSGD_OK;
    if (!seen || !first) return AQSGD_ERR_NULL;
    if (!aligned(first, 4) || !aligned(seen, 4)) return AQSGD_ERR_ALIGN;
    SeenArgs sa;
    sa.seen = seen; sa.first = first; sa.stamp = stamp;
    return launch_one(plan_quant(d, d->batch, d->n_per, act, sample_ids, m_buf, codes, scales, sa),
                      static_cast<hipStream_t>(stream));
}

int aqsgd_decode_seen(const aqsgd_desc* d, const uint8_t* codes, const float* scales, const void* full,
                      const int64_t* sample_ids, void* m_buf, uint32_t* seen, uint32_t stamp, void* out,
                      void* stream) {
    const int rc = check_decode(d, codes, scales, sample_ids, m_buf, out);
    if (rc != AQSGD_OK) return rc;
    if (stamp == 0) return AQSGD_ERR_SHAPE;
    if (d->batch == 0) return AQSGD_OK;
    if (!seen || !full) return AQSGD_ERR_NULL;
    if (!aligned(full, 16) || !aligned(seen, 4)) return AQSGD_ERR_ALIGN;
    SeenArgs sa;
    sa.seen = seen; sa.full = full; sa.stamp = stamp;
    return launch_one(plan_dequant(d, d->batch, d->n_per, codes, scales, sample_ids, m_buf, out, sa),
                      static_cast<hipStream_t>(stream));
}

size_t aqsgd_lowbit_row_bytes(const aqsgd_desc* d, int32_t m_bits) {
    if (check_lowbit(d, m_bits) != AQSGD_OK) return 0;
    return static_cast<size_t>(d->n_per) * m_bits / 8;
}

int aqsgd_encode_lowbit(const aqsgd_desc* d, int32_t m_bits, const void* act, const int64_t* sample_ids,
                        uint8_t* m_codes, float* m_scales, uint8_t* codes, float* scales, void* stream) {
    const int rc = check_lowbit(d, m_bits);
    if (rc != AQSGD_OK) return rc;
    if (d->batch == 0) return AQSGD_OK;
    if (!act || !sample_ids || !m_codes || !m_scales || !codes || !scales) return AQSGD_ERR_NULL;
    if (!aligned(act, 16) || !aligned(m_codes, 16) || !aligned(codes, 16) || !aligned(scales, 4) ||
        !aligned(m_scales, 4) || !aligned(sample_ids, 8))
        return AQSGD_ERR_ALIGN;
    return run_lowbit(d, m_bits, true, act, nullptr, sample_ids, m_codes, m_scales, codes, scales,
                      static_cast<hipStream_t>(stream));
}

int aqsgd_decode_lowbit(const aqsgd_desc* d, int32_t m_bits, const uint8_t* codes, const float* scales,
                        const int64_t* sample_ids, uint8_t* m_codes, float* m_scales, void* out,
                        void* stream) {
    const int rc = check_lowbit(d, m_bits);
    if (rc != AQSGD_OK) return rc;
    if (d->batch == 0) return AQSGD_OK;
    if (!codes || !scales || !sample_ids || !m_codes || !m_scales || !out) return AQSGD_ERR_NULL;
    if (!aligned(out, 16) || !aligned(m_codes, 16) || !aligned(codes, 16) || !aligned(scales, 4) ||
        !aligned(m_scales, 4) || !aligned(sample_ids, 8))
        return AQSGD_ERR_ALIGN;
    return run_lowbit(d, m_bits, false, nullptr, out, sample_ids, m_codes, m_scales,
                      const_cast<uint8_t*>(codes), const_cast<float*>(scales), static_cast<hipStream_t>(stream));
}

size_t aqsgd_topk_bitmap_bytes(const aqsgd_desc* d) {
    if (check_topk(d, 1) != AQSGD_OK) return 0;
    return static_cast<size_t>(d->batch) * static_cast<size_t>(d->n_per) / 8;
}

size_t aqsgd_topk_codes_bytes(const aqsgd_desc* d, int32_t keep) {
    if (check_topk(d, keep) != AQSGD_OK) return 0;
    return static_cast<size_t>(d->batch) * static_cast<size_t>(d->n_per / d->group) * keep;
}

int aqsgd_grad_topk_quant(const aqsgd_desc* d, int32_t keep, const void* grad, uint8_t* bitmap,
                          uint8_t* codes, float* scales, void* stream) {
    const int rc = check_topk(d, keep);
    if (rc != AQSGD_OK) return rc;
    if (d->batch == 0) return AQSGD_OK;
    if (!grad || !bitmap || !codes || !scales) return AQSGD_ERR_NULL;
    if (!aligned(grad, 16) || !aligned(scales, 4) || (keep % 16 == 0 && !aligned(codes, 16)))
        return AQSGD_ERR_ALIGN;
    return run_topk(d, keep, true, grad, nullptr, bitmap, codes, scales, static_cast<hipStream_t>(stream));
}

int aqsgd_grad_topk_dequant(const aqsgd_desc* d, int32_t keep, const uint8_t* bitmap, const uint8_t* codes,
                            const float* scales, void* out, void* stream) {
    const int rc = check_topk(d, keep);
    if (rc != AQSGD_OK) return rc;
    if (d->batch == 0) return AQSGD_OK;
    if (!bitmap || !codes || !scales || !out) return AQSGD_ERR_NULL;
    if (!aligned(out, 16) || !aligned(scales, 4) || (keep % 16 == 0 && !aligned(codes, 16)))
        return AQSGD_ERR_ALIGN;
    return run_topk(d, keep, false, nullptr, out, const_cast<uint8_t*>(bitmap), const_cast<uint8_t*>(codes),
                    const_cast<float*>(scales), static_cast<hipStream_t>(stream));
}

int aqsgd_check_ids(const int64_t* sample_ids, int64_t batch, int64_t n_samples, int32_t* flag,
                    void* stream) {
    if (batch < 0 || n_samples < 0) return AQSGD_ERR_SHAPE;
    if (batch == 0) return AQSGD_OK;
    if (!sample_ids || !flag) return AQSGD_ERR_NULL;
    if (!aligned(sample_ids, 8) || !aligned(flag, 4)) return AQSGD_ERR_ALIGN;
    const int64_t blocks = (batch + kBlock - 1) / kBlock;
    const hipError_t err = launch_kernel(check_ids_kernel, dim3(static_cast<unsigned>(blocks < 1024 ? blocks : 1024)),
                                         dim3(kBlock), static_cast<hipStream_t>(stream), sample_ids, batch,
                                         n_samples, flag);
    return err == hipSuccess ? AQSGD_OK : AQSGD_ERR_LAUNCH;
}

int aqsgd_set_launch_shape(int64_t max_blocks, int32_t dequant_unroll) {
    if (max_blocks < 0 || max_blocks >= (int64_t{1} << 30)) return AQSGD_ERR_SHAPE;
    if (dequant_unroll != 0 && dequant_unroll != 1 && dequant_unroll != 2 && dequant_unroll != 4)
        return AQSGD_ERR_SHAPE;
    max_blocks_knob().store(max_blocks ? max_blocks : env_max_blocks(), std::memory_order_relaxed);
    dequant_unroll_knob().store(dequant_unroll ? dequant_unroll : env_dequant_unroll(),
                                std::memory_order_relaxed);
    return AQSGD_OK;
}

int aqsgd_profile_next_launch(void* start_event, void* stop_event) {
    g_profile_request.start = static_cast<hipEvent_t>(start_event);
    g_profile_request.stop = static_cast<hipEvent_t>(stop_event);
    return AQSGD_OK;
}

const char* aqsgd_strerror(int status) {
    switch (status) {
    case AQSGD_OK:         return "ok";
    case AQSGD_ERR_NULL:   return "a required pointer is NULL";
    case AQSGD_ERR_BITS:   return "bits must be 2, 3, 4, 6 or 8";
    case AQSGD_ERR_GROUP:  return "group must be positive, divide n_per, and hold whole bytes of codes";
    case AQSGD_ERR_DTYPE:  return "unknown dtype or rounding mode";
    case AQSGD_ERR_SHAPE:  return "a size, count, stamp or slot is negative, zero, too large or out of turn";
    case AQSGD_ERR_ALIGN:  return "a pointer misses its required alignment";
    case AQSGD_ERR_LAUNCH: return "the HIP runtime refused the kernel launch, or host memory ran out";
    case AQSGD_ERR_IO:     return "the file tier could not open, size, read or write its file";
    default:               return "unknown status";
    }
}

const char* aqsgd_version(void) { return "0.1.0"; }

}  // extern "C"
