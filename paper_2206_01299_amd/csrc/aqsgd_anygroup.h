// Kernels for groups outside the job kernels' range (one message per launch):
//
//   odd groups    8 elements or more but no whole number of chunks: the flat dequantising
//                 body whose last chunk of a group stores only the elements that are its
//                 own (the quantising side is the team bodies with ODD offsets, launched
//                 from aqsgd_single.h)
//   large groups  more than a workgroup's registers hold (over 32768 elements): the maximum
//                 is taken by many workgroups into the message's scale word, and a second
//                 pass over the same elements quantises with it
//
// All of them access 16 bytes per lane at any element's address.
#pragma once

#include "aqsgd_kernels.h"
#include "aqsgd_single.h"

namespace aqsgd {

// ---------------------------------------------------------------------------
// One 16-byte piece of elements (eight, or four of binary32) and its codes, at any address.
// A 3-bit piece of four would not be whole bytes: binary32 takes eight there.
// ---------------------------------------------------------------------------
template <int DT, int BITS> struct Piece {
    static constexpr int elems = DT == AQSGD_F32 && BITS != 3 ? 4 : 8;
    static constexpr int code_bytes = elems * BITS / 8;
};

// The last `own` of the piece's elements (the others belong to the piece before it).
template <int DT, int N>
__device__ __forceinline__ void store_last_elems(void* base, int64_t at, const float (&v)[N], int own) {
#pragma unroll
    for (int e = 0; e < N; ++e)
        if (e >= N - own) store_elem<DT>(base, at + e, v[e]);
}

template <int DT, int N>
__device__ __forceinline__ void load_piece(const char* p, float (&v)[N]) {
    if constexpr (DT == AQSGD_F32) {
#pragma unroll
        for (int q = 0; q < N / 4; ++q) {
            const f32x4_t x = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any_t*>(p + 16 * q));
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * q + e] = x[e];
        }
    } else {
        unpack_raw<DT>(load_raw_any<DT>(p), v);
    }
}
template <int DT, int N>
__device__ __forceinline__ void store_piece(char* p, const float (&v)[N]) {
    if constexpr (DT == AQSGD_F32) {
#pragma unroll
        for (int q = 0; q < N / 4; ++q)
            store16_through(p + 16 * q, f32x4_t{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]});
    } else {
        store16_through(p, pack_raw<DT>(v).v);
    }
}

// Levels of a piece to / from its code word.
template <int BITS, int N>
__device__ __forceinline__ uint64_t pack_piece(const float (&q)[N]) {
    float x[kChunk];
#pragma unroll
    for (int e = 0; e < kChunk; ++e) x[e] = e < N ? q[e < N ? e : 0] : 0.0f;
    return pack_levels<BITS>(x);
}
template <int BITS, int N>
__device__ __forceinline__ void unpack_piece(uint64_t w, float (&q)[N]) {
    float x[kChunk];
    unpack_levels<BITS>(w, x);
#pragma unroll
    for (int e = 0; e < N; ++e) q[e] = x[e];
}

// ---------------------------------------------------------------------------
// Odd groups, dequantising side: flat over the pieces of a sample, UNROLL per lane and
// step, all loads first.  With previous messages the pieces of a group must not overlap
// in what they store (another wave may already have updated the shared elements), so a
// group's last piece stores its own elements one by one.
// ---------------------------------------------------------------------------
constexpr int kOddUnroll = 2;
constexpr int64_t kMaxOddPieces = int64_t{1} << 31;      // pieces of a sample: 32-bit indices with room for a step

template <int DT, int BITS, bool HAS_BUF, bool LOOPS>
__device__ __forceinline__ void dequant_odd_body(const DequantJob& a) {
    using P = Piece<DT, BITS>;
    constexpr int N = P::elems;
    constexpr int kEB = ElemBytes<DT>::value;
    constexpr uint32_t kStep = kBlock * kOddUnroll;
    const uint32_t ppg = (static_cast<uint32_t>(a.group) + N - 1) / N;           // pieces per group
    const float rcp_ppg = 1.0f / static_cast<float>(ppg);
    const uint32_t pps = static_cast<uint32_t>(a.gps) * ppg;                     // pieces per sample
    const uint32_t last_at = static_cast<uint32_t>(a.group) - N;                 // first element of a group's last piece
    const int own_last = a.group - N * static_cast<int>(ppg - 1);
    for (int i = blockIdx.y; !LOOPS || i < a.batch; i += a.grid_y) {
        const int64_t row = a.ids ? sample_id(a.ids, i) : static_cast<int64_t>(i);
        const int64_t out0 = static_cast<int64_t>(i) * a.n_per;
        char* out_s = static_cast<char*>(a.out) + out0 * kEB;
        char* m_s = HAS_BUF ? static_cast<char*>(a.m_buf) + row * a.n_per * kEB : nullptr;
        const uint8_t* codes_s = a.codes + out0 * BITS / 8;
        const float* scales_s = a.scales + static_cast<int64_t>(i) * a.gps;

        bool fresh = false;
        if constexpr (HAS_BUF) {
            if (a.seen != nullptr) {
                fresh = __builtin_amdgcn_readfirstlane(first_visit(a.seen, row, a.stamp) ? 1 : 0) != 0;
                if (fresh && blockIdx.x == 0 && threadIdx.x == 0) a.seen[row] = a.stamp;   // one writer per sample
            }
        }
        for (uint32_t base = blockIdx.x * kStep; !LOOPS || base < pps; base += a.grid_x * kStep) {
            const uint32_t g0 = base / ppg;              // uniform; per lane a small correction
            const uint32_t r0 = base - g0 * ppg;
            uint64_t w[kOddUnroll];
            float scale[kOddUnroll], m[kOddUnroll][N];
            int64_t at[kOddUnroll];                      // the piece's first element in the sample
            bool ok[kOddUnroll], last[kOddUnroll];
#pragma unroll
            for (int u = 0; u < kOddUnroll; ++u) {
                const uint32_t p = base + u * kBlock + threadIdx.x;
                ok[u] = p < pps;
                const uint32_t x = r0 + ((ok[u] ? p : pps - 1) - base);
                uint32_t dg;
                if (ppg >= kStep) {
                    dg = x >= ppg ? 1u : 0u;
                } else {                                 // x < 2^23: float is exact enough
                    dg = static_cast<uint32_t>(static_cast<float>(x) * rcp_ppg);
                    if (dg * ppg > x) --dg;
                    else if ((dg + 1) * ppg <= x) ++dg;
                }
                const uint32_t k = x - dg * ppg;         // piece within its group
                last[u] = k == ppg - 1;
                const uint32_t in_group = last[u] ? last_at : k * N;
                const int64_t g = static_cast<int64_t>(g0) + dg;
                at[u] = g * a.group + in_group;
                if (fresh) {
                    load_piece<DT, N>(static_cast<const char*>(a.full) + (out0 + at[u]) * kEB, m[u]);
                    continue;
                }
                w[u] = load_bytes_any<P::code_bytes>(codes_s + (g * a.group * BITS / 8 + in_group * BITS / 8));
                scale[u] = scales_s[g];
                if constexpr (HAS_BUF) load_piece<DT, N>(m_s + at[u] * kEB, m[u]);
            }
            __builtin_amdgcn_sched_barrier(0);           // every load is out before the first use
#pragma unroll
            for (int u = 0; u < kOddUnroll; ++u) {
                if (!ok[u]) continue;
                if (fresh) {                             // the uncompressed row; repeated elements repeat their value
                    store_piece<DT, N>(m_s + at[u] * kEB, m[u]);
                    store_piece<DT, N>(out_s + at[u] * kEB, m[u]);
                    continue;
                }
                const GroupScale sc = scale_from_wire<BITS>(scale[u]);
                float v[N];
                unpack_piece<BITS, N>(w[u], v);
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    v[e] = value_of(v[e], sc);
                    if constexpr (HAS_BUF) v[e] = m[u][e] + v[e];
                }
                if (HAS_BUF && last[u]) {
                    store_last_elems<DT, N>(m_s, at[u], v, own_last);
                    store_last_elems<DT, N>(out_s, at[u], v, own_last);
                } else {
                    if constexpr (HAS_BUF) store_piece<DT, N>(m_s + at[u] * kEB, v);
                    store_piece<DT, N>(out_s + at[u] * kEB, v);
                }
            }
            if constexpr (!LOOPS) break;
        }
        if constexpr (!LOOPS) break;
    }
}

template <int DT, int BITS, bool LOOPS>
__device__ __forceinline__ void dequant_odd_bits(const DequantJob& a) {
    if (a.m_buf) dequant_odd_body<DT, BITS, true, LOOPS>(a);
    else dequant_odd_body<DT, BITS, false, LOOPS>(a);
}

template <int DT, bool LOOPS>
__global__ __launch_bounds__(kBlock)
void dequant_odd_kernel(AQSGD_DEQUANT_ARGS) {
    DequantJob a;
    a.codes = codes; a.scales = scales; a.ids = ids; a.m_buf = m_buf; a.out = out; a.full = full;
    a.n_per = n_per; a.gps = gps; a.batch = batch; a.group = group; a.bits = bits;
    a.grid_x = grid_x; a.grid_y = grid_y;
    a.seen = seen; a.stamp = stamp;
    switch (bits) {
    case 2: dequant_odd_bits<DT, 2, LOOPS>(a); break;
    case 4: dequant_odd_bits<DT, 4, LOOPS>(a); break;
    case 6: dequant_odd_bits<DT, 6, LOOPS>(a); break;
    default: dequant_odd_bits<DT, 8, LOOPS>(a); break;
    }
}

// ---------------------------------------------------------------------------
// Large groups, quantising side: three launches.  The message's scale word of a group
// collects the maximum (magnitudes order like unsigned integers, and any order of an
// atomic maximum gives the same bits), so no memory beyond the call's own is needed:
//   1. the scale words are cleared
//   2. every workgroup takes the maximum of its span of a group into the group's word
//   3. the same spans are read again, quantised with the finished word and stored
// A group's spans are read twice, the second time mostly from the last-level cache.
// (bfloat16, eight samples with one scale each, 49152 elements, forward and backward in
// four calls: one thread per group 31.9 ms, now 47 us.)
// ---------------------------------------------------------------------------
struct LargeGeom {
    int32_t spans;             // spans per group
    int32_t span_pieces;       // pieces of 8 elements per span: a multiple of kBlock
};

constexpr int kLargeUnroll = 4;                          // pieces per lane and step
constexpr int64_t kLargeMinSpanPieces = static_cast<int64_t>(kBlock) * kLargeUnroll;
constexpr int64_t kLargeMaxBlocks = 2048;                // about what is resident at once

template <bool HAS_BUF>
__device__ __forceinline__ bool large_fresh(const QuantJob& a, int64_t row) {
    if constexpr (HAS_BUF)
        return a.seen != nullptr &&
               __builtin_amdgcn_readfirstlane(first_visit(a.seen, row, a.stamp) ? 1 : 0) != 0;
    else return false;
}

static __global__ __launch_bounds__(kBlock)
void large_clear_kernel(const QuantJob a) {
    for (int i = blockIdx.y; i < a.batch; i += gridDim.y) {
        const int64_t row = a.ids ? sample_id(a.ids, i) : static_cast<int64_t>(i);
        if (large_fresh<true>(a, row)) continue;         // a new sample's scales are not written
        for (int64_t g = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; g < a.gps;
             g += static_cast<int64_t>(gridDim.x) * kBlock)
            a.scales[static_cast<int64_t>(i) * a.gps + g] = 0.0f;
    }
}

template <int DT, bool HAS_BUF>
__device__ __forceinline__ void large_max_body(const QuantJob& a, const LargeGeom geom, float* wave_max) {
    constexpr int N = DT == AQSGD_F32 ? 4 : 8;
    constexpr int kEB = ElemBytes<DT>::value;
    const int64_t last_at = a.group - N;
    for (int i = blockIdx.y; i < a.batch; i += gridDim.y) {
        const int64_t row = a.ids ? sample_id(a.ids, i) : static_cast<int64_t>(i);
        if (large_fresh<HAS_BUF>(a, row)) continue;
        const char* src_s = static_cast<const char*>(a.src) + static_cast<int64_t>(i) * a.n_per * kEB;
        const char* m_s = HAS_BUF ? static_cast<const char*>(a.m_buf) + row * a.n_per * kEB : nullptr;
        for (int64_t s = blockIdx.x; s < a.gps * geom.spans; s += gridDim.x) {
            const int64_t g = s / geom.spans;
            const int64_t e0 = (s - g * geom.spans) * geom.span_pieces * 8;
            const int64_t e1 = min(e0 + static_cast<int64_t>(geom.span_pieces) * 8, static_cast<int64_t>(a.group));
            const char* src_g = src_s + g * a.group * kEB;
            const char* m_g = HAS_BUF ? m_s + g * a.group * kEB : nullptr;
            float mx = 0.0f;
            for (int64_t e = e0 + static_cast<int64_t>(threadIdx.x) * N; e < e1;
                 e += static_cast<int64_t>(kBlock) * N * kLargeUnroll) {
                float x[kLargeUnroll][N], m[kLargeUnroll][N];
#pragma unroll
                for (int u = 0; u < kLargeUnroll; ++u) { // past the end: the group's last piece once more
                    const int64_t at = min(e + static_cast<int64_t>(u) * kBlock * N, last_at);
                    load_piece<DT, N>(src_g + at * kEB, x[u]);
                    if constexpr (HAS_BUF) load_piece<DT, N>(m_g + at * kEB, m[u]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kLargeUnroll; ++u)
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        const float d = HAS_BUF ? x[u][k] - m[u][k] : x[u][k];
                        mx = __builtin_fmaxf(mx, __builtin_fabsf(d));
                    }
            }
            mx = team_max<kWave>(mx);
            __syncthreads();                             // earlier readers of wave_max are done
            if (threadIdx.x % kWave == 0) wave_max[threadIdx.x / kWave] = mx;
            __syncthreads();
            if (threadIdx.x == 0) {
#pragma unroll
                for (int w = 0; w < kBlock / kWave; ++w) mx = __builtin_fmaxf(mx, wave_max[w]);
                atomicMax(reinterpret_cast<unsigned int*>(a.scales) + static_cast<int64_t>(i) * a.gps + g,
                          __float_as_uint(mx));
            }
        }
    }
}

template <int DT>
__global__ __launch_bounds__(kBlock)
void large_max_kernel(const QuantJob a, const LargeGeom geom) {
    __shared__ float wave_max[kBlock / kWave];
    if (a.m_buf) large_max_body<DT, true>(a, geom, wave_max);
    else large_max_body<DT, false>(a, geom, wave_max);
}

// A group below the 2^-120 floor sends scale 0; one thread rewrites its word while other
// workgroups may still read it, and both values mean "nothing to send" to them.
template <int DT, int BITS, int ROUND, bool HAS_BUF>
__device__ __forceinline__ void large_quant_body(const QuantJob& a, const LargeGeom geom) {
    using P = Piece<DT, BITS>;
    constexpr int N = P::elems;
    constexpr int kEB = ElemBytes<DT>::value;
    const int64_t last_at = a.group - N;
    for (int i = blockIdx.y; i < a.batch; i += gridDim.y) {
        const int64_t row = a.ids ? sample_id(a.ids, i) : static_cast<int64_t>(i);
        const int64_t src0 = static_cast<int64_t>(i) * a.n_per;
        const char* src_s = static_cast<const char*>(a.src) + src0 * kEB;
        char* m_s = HAS_BUF ? static_cast<char*>(a.m_buf) + row * a.n_per * kEB : nullptr;
        const bool fresh = large_fresh<HAS_BUF>(a, row);
        if constexpr (HAS_BUF) {
            if (a.seen != nullptr && blockIdx.x == 0 && threadIdx.x == 0) {      // one writer per sample
                a.first[i] = fresh ? 1 : 0;
                if (fresh) a.seen[row] = a.stamp;
            }
        }
        for (int64_t s = blockIdx.x; s < a.gps * geom.spans; s += gridDim.x) {
            const int64_t g = s / geom.spans;
            const int64_t e0 = (s - g * geom.spans) * geom.span_pieces * 8;
            const int64_t e1 = min(e0 + static_cast<int64_t>(geom.span_pieces) * 8, static_cast<int64_t>(a.group));
            const int64_t goff = g * a.group;
            const char* src_g = src_s + goff * kEB;
            char* m_g = HAS_BUF ? m_s + goff * kEB : nullptr;
            uint8_t* codes_g = a.codes + (src0 + goff) * BITS / 8;
            float* const word = a.scales + static_cast<int64_t>(i) * a.gps + g;
            GroupScale sc;
            if (!fresh) {
                sc = make_scale<BITS>(*word);
                if (e0 == 0 && threadIdx.x == 0 && sc.s_tx == 0.0f) *word = 0.0f;
            }
            for (int64_t e = e0 + static_cast<int64_t>(threadIdx.x) * N; e < e1;
                 e += static_cast<int64_t>(kBlock) * N * kLargeUnroll) {
                float x[kLargeUnroll][N], m[kLargeUnroll][N];
                int64_t at[kLargeUnroll];
#pragma unroll
                for (int u = 0; u < kLargeUnroll; ++u) {
                    at[u] = min(e + static_cast<int64_t>(u) * kBlock * N, last_at);
                    load_piece<DT, N>(src_g + at[u] * kEB, x[u]);
                    if constexpr (HAS_BUF) load_piece<DT, N>(m_g + at[u] * kEB, m[u]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kLargeUnroll; ++u) {
                    const int64_t eu = e + static_cast<int64_t>(u) * kBlock * N;
                    if (eu >= e1) continue;
                    // the group's last piece owns what the one before it does not
                    const int own = static_cast<int>(min(static_cast<int64_t>(N), a.group - eu));
                    if (fresh) {
                        if constexpr (HAS_BUF) store_piece<DT, N>(m_g + at[u] * kEB, x[u]);
                        continue;
                    }
                    float r[N], q[N], v[N];
                    if constexpr (ROUND == AQSGD_ROUND_STOCHASTIC) {
                        uniforms_any<N>(a.seed, static_cast<uint64_t>(src0 + goff + at[u]), r);
                    } else {
#pragma unroll
                        for (int k = 0; k < N; ++k) r[k] = kNearestOffset32;
                    }
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        const float d = HAS_BUF ? x[u][k] - m[u][k] : x[u][k] - 0.0f;
                        q[k] = level_of<BITS, ROUND>(d, sc, r[k]);
                        v[k] = value_of(q[k], sc);
                        if constexpr (HAS_BUF) v[k] = m[u][k] + v[k];
                    }
                    const uint64_t w = pack_piece<BITS, N>(q);
                    uint8_t* c = codes_g + at[u] * BITS / 8;
                    if (own == N) {
                        store_bytes_any<P::code_bytes>(c, w);
                        if constexpr (HAS_BUF) store_piece<DT, N>(m_g + at[u] * kEB, v);
                    } else {
                        const int skip = (N - own) * BITS / 8;                   // whole bytes, as the group's are
                        for (int b = skip; b < P::code_bytes; ++b) c[b] = static_cast<uint8_t>(w >> (8 * b));
                        if constexpr (HAS_BUF) store_last_elems<DT, N>(m_g, at[u], v, own);
                    }
                }
            }
        }
    }
}

template <int DT, int BITS, int ROUND>
__device__ __forceinline__ void large_quant_bits(const QuantJob& a, const LargeGeom geom) {
    if (a.m_buf) large_quant_body<DT, BITS, ROUND, true>(a, geom);
    else large_quant_body<DT, BITS, ROUND, false>(a, geom);
}

template <int DT, int ROUND>
__global__ __launch_bounds__(kBlock)
void large_quant_kernel(const QuantJob a, const LargeGeom geom) {
    switch (a.bits) {
    case 2: large_quant_bits<DT, 2, ROUND>(a, geom); break;
    case 3: large_quant_bits<DT, 3, ROUND>(a, geom); break;
    case 4: large_quant_bits<DT, 4, ROUND>(a, geom); break;
    case 6: large_quant_bits<DT, 6, ROUND>(a, geom); break;
    default: large_quant_bits<DT, 8, ROUND>(a, geom); break;
    }
}

// Per-dtype pieces (defined by AQSGD_INSTANTIATE_ANYGROUP_DTYPE in the dtype's .hip file).
template <int DT> hipError_t launch_dequant_odd_dt(bool covers, const DequantJob& a, hipStream_t stream);
template <int DT> hipError_t launch_quant_large_dt(int rounding, const QuantJob& a, const LargeGeom& geom,
                                                   hipStream_t stream);

// ---- launch tables (instantiated per dtype in aqsgd_anygroup_<dtype>.hip) --------------
template <int DT>
hipError_t launch_dequant_odd_dt(bool covers, const DequantJob& a, hipStream_t s) {
    return covers ? launch_dequant_with(dequant_odd_kernel<DT, false>, a, s)
                  : launch_dequant_with(dequant_odd_kernel<DT, true>, a, s);
}

template <int DT>
hipError_t launch_quant_large_dt(int rounding, const QuantJob& a, const LargeGeom& geom, hipStream_t s) {
    const int64_t clear_x = (a.gps + kBlock - 1) / kBlock;
    const dim3 grid(a.grid_x, a.grid_y), block(kBlock);
    hipError_t err = launch_kernel(large_clear_kernel, dim3(static_cast<unsigned>(clear_x < 1024 ? clear_x : 1024), a.grid_y),
                                   block, s, a);
    if (err == hipSuccess) err = launch_kernel(large_max_kernel<DT>, grid, block, s, a, geom);
    if (err == hipSuccess)
        err = rounding == AQSGD_ROUND_STOCHASTIC
                  ? launch_kernel(large_quant_kernel<DT, AQSGD_ROUND_STOCHASTIC>, grid, block, s, a, geom)
                  : launch_kernel(large_quant_kernel<DT, AQSGD_ROUND_NEAREST>, grid, block, s, a, geom);
    return err;
}

#define AQSGD_INSTANTIATE_ANYGROUP_DTYPE(DT)                                                          \
    template hipError_t launch_dequant_odd_dt<DT>(bool, const DequantJob&, hipStream_t);                   \
    template hipError_t launch_quant_large_dt<DT>(int, const QuantJob&, const LargeGeom&, hipStream_t);

}  // namespace aqsgd
