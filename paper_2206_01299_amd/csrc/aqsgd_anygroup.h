// Kernels for groups outside the job kernels' range, a message a launch, and the bodies that the shared
// launches of such messages are made of (aqsgd_jobs_anygroup.h):
//
//   odd groups    8 elements or more but no whole number of chunks: a flat dequantising
//                 body whose pieces may hold the end of one group and the start of the
//                 next (the quantising side is the team bodies with ODD offsets; alone
//                 they are launched from aqsgd_single.h)
//   wide groups   more elements than the job kernels' shapes take (over 32768) that one
//                 workgroup still holds in registers as stored: one pass
//   large groups  more than that: the maximum is taken by many workgroups into the
//                 message's scale word, and a second pass over the same elements quantises
//                 with it
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
__device__ __forceinline__ void store_piece(char* p, const float (&v)[N], bool through = false) {
    if constexpr (DT == AQSGD_F32) {
#pragma unroll
        for (int q = 0; q < N / 4; ++q)
            store16(p + 16 * q, f32x4_t{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]}, through);
    } else {
        store16(p, pack_raw<DT>(v).v, through);
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
// Odd groups, dequantising side: flat over the 16-byte pieces of a sample, UNROLL per lane and
// step, all loads first.  The codes of a sample are one bit stream whatever its groups, so a piece
// starts at a multiple of its length (aligned, wherever rows are whole pieces) and only its scale
// changes inside it, at most once in eight elements.  Pieces that start with every group instead
// sit at odd addresses, and the last one of a group has to store its own elements one by one where
// previous messages are updated in place: decode of float16 [2,2048,942] 9.1 us that way and 6.5
// this, [16,400,102] 5.2 and 3.9, grad_dequant of [4,250,1020] 3.6 and 3.2.  Only a sample that is
// no whole number of pieces ends in such a piece here.
//
// SEAMS: a piece may hold two groups.  float32 groups of whole pieces have none, and a body that looks
// for them costs a grad_dequant a tenth: [8,500,1020] pieces that start with every group 4.29 us, with
// seams 4.86, without 4.05; [8,1000,1020] 6.46, 7.28, 6.30.
// ---------------------------------------------------------------------------
constexpr int kOddUnroll = 2;
constexpr int64_t kMaxOddPieces = int64_t{1} << 31;      // pieces of a sample: 32-bit indices with room for a step

template <int DT, int BITS, bool HAS_BUF, bool SEAMS, int THREADS, bool LOOPS, bool THROUGH = false>
__device__ __forceinline__ void dequant_odd_body(const DequantJob& a, uint32_t bx, uint32_t by) {
    using P = Piece<DT, BITS>;
    constexpr int N = P::elems;
    constexpr int kEB = ElemBytes<DT>::value;
    constexpr uint32_t kStep = THREADS * kOddUnroll;
    const uint32_t group = static_cast<uint32_t>(a.group);
    // one Newton step brings the estimate of 1 / group well below the 2^-32 that a quotient needs
    const double estimate = __builtin_amdgcn_rcp(static_cast<double>(a.group));
    const double rcp_group = __builtin_fma(__builtin_fma(-static_cast<double>(a.group), estimate, 1.0), estimate, estimate);
    const float rcp_small = static_cast<float>(rcp_group);
    const uint32_t pps = static_cast<uint32_t>((a.n_per + N - 1) / N);   // pieces per sample: below 2^31, checked by the host
    const int rest = static_cast<int>(a.n_per % N);                      // elements of a last piece that is no whole one
    for (int i = by; !LOOPS || i < a.batch; i += a.grid_y) {
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
                if (fresh && bx == 0 && threadIdx.x == 0) a.seen[row] = a.stamp;   // one writer per sample
            }
        }
        for (uint32_t base = bx * kStep; !LOOPS || base < pps; base += a.grid_x * kStep) {
            // group of the step's first element (uniform): the quotient is off by one at most
            const int64_t e0 = static_cast<int64_t>(base) * N;
            int64_t g0 = static_cast<int64_t>(static_cast<double>(e0) * rcp_group);
            if (g0 * a.group > e0) --g0;
            else if ((g0 + 1) * a.group <= e0) ++g0;
            const uint32_t r0 = static_cast<uint32_t>(e0 - g0 * a.group);
            uint64_t w[kOddUnroll];
            float scale[kOddUnroll], next_scale[kOddUnroll], m[kOddUnroll][N];
            int64_t at[kOddUnroll];                      // the piece's first element in the sample
            int left[kOddUnroll];                        // elements of its group from there on
            bool ok[kOddUnroll], last[kOddUnroll];
#pragma unroll
            for (int u = 0; u < kOddUnroll; ++u) {
                const uint32_t p = base + u * THREADS + threadIdx.x;
                ok[u] = p < pps;
                const uint32_t piece = ok[u] ? p : pps - 1;
                const uint32_t x = r0 + (piece - base) * N;
                uint32_t dg;
                if (group >= kStep * N) {
                    dg = x >= group ? 1u : 0u;
                } else {                                 // x < 2^17: float is exact enough
                    dg = static_cast<uint32_t>(static_cast<float>(x) * rcp_small);
                    if (dg * group > x) --dg;
                    else if ((dg + 1) * group <= x) ++dg;
                }
                last[u] = SEAMS && rest != 0 && piece == pps - 1;         // ends with the sample, and with its group
                at[u] = last[u] ? a.n_per - N : static_cast<int64_t>(piece) * N;
                left[u] = last[u] ? N : static_cast<int>(group - (x - dg * group));
                if (fresh) {
                    load_piece<DT, N>(static_cast<const char*>(a.full) + (out0 + at[u]) * kEB, m[u]);
                    continue;
                }
                w[u] = load_bytes_any<P::code_bytes>(codes_s + static_cast<uint64_t>(at[u]) * BITS / 8);   // whole bytes
                const float* s = scales_s + (g0 + dg);
                scale[u] = s[0];
                if constexpr (SEAMS) next_scale[u] = s[left[u] < N ? 1 : 0];
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
                const GroupScale here = scale_from_wire<BITS>(scale[u]);
                [[maybe_unused]] GroupScale next;
                if constexpr (SEAMS) next = scale_from_wire<BITS>(next_scale[u]);
                float v[N];
                unpack_piece<BITS, N>(w[u], v);
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    GroupScale sc = here;
                    if constexpr (SEAMS) {
                        sc.offset = e < left[u] ? here.offset : next.offset;
                        sc.step = e < left[u] ? here.step : next.step;
                    }
                    v[e] = value_of(v[e], sc);
                    if constexpr (HAS_BUF) v[e] = m[u][e] + v[e];
                }
                if (last[u]) {                           // the elements before are another piece's, and may be updated by now
                    if constexpr (HAS_BUF) store_last_elems<DT, N>(m_s, at[u], v, rest);
                    store_last_elems<DT, N>(out_s, at[u], v, rest);
                } else {
                    if constexpr (HAS_BUF) store_piece<DT, N>(m_s + at[u] * kEB, v);
                    store_piece<DT, N>(out_s + at[u] * kEB, v, THROUGH);
                }
            }
            if constexpr (!LOOPS) break;
        }
        if constexpr (!LOOPS) break;
    }
}

template <int DT, int BITS, int THREADS, bool LOOPS>
__device__ __forceinline__ void dequant_odd_bits(const DequantJob& a, uint32_t bx, uint32_t by) {
    if constexpr (Piece<DT, BITS>::elems < kChunk) {     // float32: groups of whole pieces, without seams
        if (a.group % Piece<DT, BITS>::elems == 0) {     // uniform over the workgroup
            if (a.m_buf) dequant_odd_body<DT, BITS, true, false, THREADS, LOOPS>(a, bx, by);
            else dequant_odd_body<DT, BITS, false, false, THREADS, LOOPS>(a, bx, by);
            return;
        }
    }
    if (a.m_buf) dequant_odd_body<DT, BITS, true, true, THREADS, LOOPS>(a, bx, by);
    else dequant_odd_body<DT, BITS, false, true, THREADS, LOOPS>(a, bx, by);
}

template <int DT, int THREADS, bool LOOPS>
__device__ __forceinline__ void dequant_odd_job(const DequantJob& a, uint32_t bx, uint32_t by) {
    switch (a.bits) {                                    // uniform over the workgroup; 3-bit groups are whole chunks
    case 2: dequant_odd_bits<DT, 2, THREADS, LOOPS>(a, bx, by); break;
    case 4: dequant_odd_bits<DT, 4, THREADS, LOOPS>(a, bx, by); break;
    case 6: dequant_odd_bits<DT, 6, THREADS, LOOPS>(a, bx, by); break;
    default: dequant_odd_bits<DT, 8, THREADS, LOOPS>(a, bx, by); break;
    }
}

// Large float32 gradients of whole pieces, which are written through the L2 (see odd_writes_through()).
template <int THREADS>
__device__ __forceinline__ void dequant_odd_through(const DequantJob& a, uint32_t bx, uint32_t by) {
    switch (a.bits) {                                    // uniform over the workgroup
    case 2: dequant_odd_body<AQSGD_F32, 2, false, false, THREADS, false, true>(a, bx, by); break;
    case 4: dequant_odd_body<AQSGD_F32, 4, false, false, THREADS, false, true>(a, bx, by); break;
    case 6: dequant_odd_body<AQSGD_F32, 6, false, false, THREADS, false, true>(a, bx, by); break;
    default: dequant_odd_body<AQSGD_F32, 8, false, false, THREADS, false, true>(a, bx, by); break;
    }
}

enum OddKind { kOddOneStep = 0, kOddLoops, kOddThrough };

template <int DT, int KIND>
__global__ __launch_bounds__(kBlock)
void dequant_odd_kernel(AQSGD_DEQUANT_ARGS) {
    DequantJob a;
    a.codes = codes; a.scales = scales; a.ids = ids; a.m_buf = m_buf; a.out = out; a.full = full;
    a.n_per = n_per; a.gps = gps; a.batch = batch; a.group = group; a.bits = bits;
    a.grid_x = grid_x; a.grid_y = grid_y;
    a.seen = seen; a.stamp = stamp;
    if constexpr (KIND == kOddThrough) dequant_odd_through<kBlock>(a, blockIdx.x, blockIdx.y);
    else dequant_odd_job<DT, kBlock, KIND == kOddLoops>(a, blockIdx.x, blockIdx.y);
}

// ---------------------------------------------------------------------------
// Wide groups, quantising side: a workgroup of 1024 lanes holds a whole group the way it is
// stored, eight 16-byte pieces of activations and eight of previous messages per lane (twelve
// in binary32), and forms the change twice, for the maximum and for the levels, instead of
// keeping it.  That is 64 (96) of the 128 registers a lane of such a workgroup has, and the
// group is read once, in one launch, where the large groups' way takes three launches and two
// readings.  All loads of a workgroup are back before its first store (the maximum waits for
// them), so a group's last piece may repeat elements of the one before it: same values, same
// results, same place.  Few groups are bound by one compute unit's arithmetic (7 to 10 us for a
// nearest encode of 49152 elements, 12 to 15 with stochastic rounding; those are split where it pays,
// see below), many by memory.  Measured as four calls on groups of 49152, large groups' way -> this:
// bfloat16, 256 groups 74 -> 48.5 us, 1024 groups 237 -> 182; float32, 256 groups 117 -> 80, 1024
// groups 431 -> 326.
// ---------------------------------------------------------------------------
constexpr int kWideThreads = 1024;
template <int DT> struct WideRounds { static constexpr int value = DT == AQSGD_F32 ? 12 : 8; };
// Rounds of a group: pieces of 16 bytes (32 of binary32 at 3 bits), one per lane and round.
constexpr int wide_rounds(int dtype, int bits, int group) {
    const int piece = dtype == AQSGD_F32 && bits != 3 ? 4 : 8;
    return ((group + piece - 1) / piece + kWideThreads - 1) / kWideThreads;
}
// Elements of the largest group: pieces of 16 bytes, one per lane and round.
constexpr int wide_most_elements(int dtype) {
    return dtype == AQSGD_F32 ? kWideThreads * 4 * WideRounds<AQSGD_F32>::value
                              : kWideThreads * 8 * WideRounds<AQSGD_F16>::value;
}

// A piece as stored.
template <int DT, int N> struct PieceRaw { u32x4_t v[N * ElemBytes<DT>::value / 16]; };

template <int DT, int N>
__device__ __forceinline__ void load_piece_raw(const char* p, PieceRaw<DT, N>& r) {
#pragma unroll
    for (int q = 0; q < N * ElemBytes<DT>::value / 16; ++q)
        r.v[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any_t*>(p + 16 * q));
}
template <int DT, int N>
__device__ __forceinline__ void piece_values(const PieceRaw<DT, N>& r, float (&f)[N]) {
    if constexpr (DT == AQSGD_F32) {
#pragma unroll
        for (int e = 0; e < N; ++e) f[e] = __uint_as_float(r.v[e / 4][e % 4]);
    } else {
        Raw<DT> x;
        x.v = r.v[0];
        unpack_raw<DT>(x, f);
    }
}

// The change of a piece, in binary32; without previous messages the values themselves.  float16
// operands are widened by the subtraction (see delta_chunk): one encode of eight groups of 49152 8.4 us
// with conversions of their own and 7.9 so.
template <int DT, int N, bool HAS_BUF>
__device__ __forceinline__ void piece_change(const PieceRaw<DT, N>& a, const PieceRaw<DT, N>& m, float (&d)[N]) {
    if constexpr (HAS_BUF && DT == AQSGD_F16) {
        delta_chunk<DT>(Raw<DT>{a.v[0]}, Raw<DT>{m.v[0]}, d);
    } else {
        piece_values<DT, N>(a, d);
        if constexpr (HAS_BUF) {
            float mv[N];
            piece_values<DT, N>(m, mv);
#pragma unroll
            for (int e = 0; e < N; ++e) d[e] = d[e] - mv[e];
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e) d[e] = d[e] - 0.0f;
        }
    }
}

// One group in a workgroup: bx is the group of the sample, by the sample.  Without previous messages
// nothing that a workgroup reads is written in the launch, so several can share a group: each takes
// the maximum of all of it and quantises `share` rounds from share * part on (few groups leave most
// compute units idle, and the levels are two thirds of the arithmetic; see wide_share() in the dispatch).
template <int DT, int BITS, int ROUND, bool HAS_BUF>
__device__ __forceinline__ void quant_wide_body(const QuantJob& a, uint32_t bx, uint32_t by, uint32_t part, int share,
                                                float* wave_max) {
    using P = Piece<DT, BITS>;
    constexpr int N = P::elems;
    constexpr int kEB = ElemBytes<DT>::value;
    constexpr int kRounds = WideRounds<DT>::value * 16 / (N * kEB);
    const int lane = threadIdx.x;
    const int rounds = ((a.group + N - 1) / N + kWideThreads - 1) / kWideThreads;    // 1 .. kRounds: checked by the host
    const int i = by;
    const int64_t g = bx;
    const int64_t row = a.ids ? sample_id(a.ids, i) : static_cast<int64_t>(i);
    bool fresh = false;
    if constexpr (HAS_BUF) {
        if (a.seen != nullptr) {
            fresh = __builtin_amdgcn_readfirstlane(first_visit(a.seen, row, a.stamp) ? 1 : 0) != 0;
            if (g == 0 && lane == 0) {                   // one writer per sample
                a.first[i] = fresh ? 1 : 0;
                if (fresh) a.seen[row] = a.stamp;
            }
        }
    }
    const int64_t src0 = static_cast<int64_t>(i) * a.n_per + g * a.group;    // the group's first element in the call
    const char* src_g = static_cast<const char*>(a.src) + src0 * kEB;
    char* m_g = HAS_BUF ? static_cast<char*>(a.m_buf) + (row * a.n_per + g * a.group) * kEB : nullptr;
    uint8_t* codes_g = a.codes + src0 * BITS / 8;
    // the first element of the lane's piece of a round
    auto place = [&](int k) {
        uint32_t at = static_cast<uint32_t>(min((k * kWideThreads + lane) * N, a.group - N));
        asm volatile("" : "+v"(at));                     // formed where it is used, not kept for every round
        return at;
    };
    PieceRaw<DT, N> ra[kRounds], rm[kRounds];
#pragma unroll
    for (int k = 0; k < kRounds; ++k)
        if (k < rounds) {                                // uniform over the launch
            const uint32_t at = place(k) * kEB;
            load_piece_raw<DT, N>(src_g + at, ra[k]);
            if constexpr (HAS_BUF) load_piece_raw<DT, N>(m_g + at, rm[k]);
        }
    __builtin_amdgcn_sched_barrier(0);
    if (fresh) {                                         // uniform over the workgroup
        __syncthreads();                                 // a repeated element is loaded before it is stored
        if constexpr (HAS_BUF) {
#pragma unroll
            for (int k = 0; k < kRounds; ++k)
                if (k < rounds) {
                    const uint32_t at = place(k) * kEB;
#pragma unroll
                    for (int q = 0; q < N * kEB / 16; ++q) store16(m_g + at + 16 * q, ra[k].v[q], false);
                }
        }
        return;
    }
    float mx = 0.0f;
#pragma unroll
    for (int k = 0; k < kRounds; ++k)
        if (k < rounds) {
            float d[N];
            piece_change<DT, N, HAS_BUF>(ra[k], rm[k], d);
#pragma unroll
            for (int e = 0; e < N; ++e) mx = __builtin_fmaxf(mx, __builtin_fabsf(d[e]));
#pragma unroll
            for (int w = 0; w < N * kEB / 16; ++w) asm volatile("" : "+v"(ra[k].v[w]));  // the change is formed again, not kept
        }
    mx = team_max<kWave>(mx);
    if (lane % kWave == 0) wave_max[lane / kWave] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWideThreads / kWave; ++w) mx = __builtin_fmaxf(mx, wave_max[w]);
    const GroupScale sc = make_scale<BITS>(mx);
    const int first = HAS_BUF ? 0 : static_cast<int>(part) * share, end = HAS_BUF ? rounds : min(first + share, rounds);
#pragma unroll
    for (int k = 0; k < kRounds; ++k)
        if (k >= first && k < end) {                     // uniform over the workgroup
            float d[N], r[N], q[N], v[N];
            const uint32_t at = place(k);
            if constexpr (ROUND == AQSGD_ROUND_STOCHASTIC) {
                if (a.group % 4 != 0) {                  // uniform over the launch
                    uniforms_any<N>(a.seed, static_cast<uint64_t>(src0) + at, r);
                } else {                                 // whole Philox blocks
#pragma unroll
                    for (int b = 0; b < N; b += 4) block_uniforms(a.seed, (static_cast<uint64_t>(src0) + at + b) >> 2, &r[b]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < N; ++e) r[e] = kNearestOffset32;
            }
            piece_change<DT, N, HAS_BUF>(ra[k], rm[k], d);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                q[e] = level_of<BITS, ROUND>(d[e], sc, r[e]);
                v[e] = value_of(q[e], sc);
            }
            store_bytes_any<P::code_bytes>(codes_g + at * BITS / 8, pack_piece<BITS, N>(q));
            if constexpr (HAS_BUF && DT == AQSGD_F16) {
                store16(m_g + at * kEB, updated_chunk<DT>(Raw<DT>{rm[k].v[0]}, v).v, false);
            } else if constexpr (HAS_BUF) {
                float m[N];
                piece_values<DT, N>(rm[k], m);
#pragma unroll
                for (int e = 0; e < N; ++e) v[e] = m[e] + v[e];
                store_piece<DT, N>(m_g + at * kEB, v);
            }
            __builtin_amdgcn_sched_barrier(0);           // one piece's temporaries at a time
        }
    if (lane == 0 && (HAS_BUF || part == 0)) a.scales[static_cast<int64_t>(i) * a.gps + g] = sc.s_tx;
}

template <int DT, int BITS, int ROUND>
__device__ __forceinline__ void quant_wide_bits(const QuantJob& a, uint32_t bx, uint32_t by, uint32_t part, int share,
                                                float* wave_max) {
    if (a.m_buf) quant_wide_body<DT, BITS, ROUND, true>(a, bx, by, part, share, wave_max);
    else quant_wide_body<DT, BITS, ROUND, false>(a, bx, by, part, share, wave_max);
}

template <int DT, int ROUND>
__device__ __forceinline__ void quant_wide_job(const QuantJob& a, uint32_t bx, uint32_t by, uint32_t part, int share,
                                               float* wave_max) {
    switch (a.bits) {                                    // uniform over the workgroup
    case 2: quant_wide_bits<DT, 2, ROUND>(a, bx, by, part, share, wave_max); break;
    case 3: quant_wide_bits<DT, 3, ROUND>(a, bx, by, part, share, wave_max); break;
    case 4: quant_wide_bits<DT, 4, ROUND>(a, bx, by, part, share, wave_max); break;
    case 6: quant_wide_bits<DT, 6, ROUND>(a, bx, by, part, share, wave_max); break;
    default: quant_wide_bits<DT, 8, ROUND>(a, bx, by, part, share, wave_max); break;
    }
}

template <int DT, int ROUND>
__global__ __launch_bounds__(kWideThreads)
void quant_wide_kernel(AQSGD_QUANT_ARGS) {
    __shared__ float wave_max[kWideThreads / kWave];
    QuantJob a;
    a.src = src; a.ids = ids; a.m_buf = m_buf; a.codes = codes; a.scales = scales;
    a.n_per = n_per; a.gps = gps; a.batch = batch; a.group = group;
    a.grid_x = grid_x; a.grid_y = grid_y;
    a.bits = bits & 255;
    a.seed = seed; a.seen = seen; a.first = first; a.stamp = stamp;
    quant_wide_job<DT, ROUND>(a, blockIdx.x, blockIdx.y, blockIdx.z, bits >> 8, wave_max);
}

// ---------------------------------------------------------------------------
// Large groups, quantising side: three launches.  The message's scale word of a group
// collects the maximum (magnitudes order like unsigned integers, and any order of an
// atomic maximum gives the same bits), so no memory beyond the call's own is needed:
//   1. the scale words are cleared
//   2. every workgroup takes the maximum of its span of a group into the group's word
//   3. the same spans are read again, quantised with the finished word and stored
// A group's spans are read twice, the second time mostly from the last-level cache.
// (bfloat16, eight groups of 49152, forward and backward in four calls: one thread per group
// 31.9 ms, this way 29.4 us.)
// ---------------------------------------------------------------------------
// The bodies rely on no more of a span's length than that the spans cover the group (the host
// rounds it to whole workgroup steps for large groups, and not for split ones).  Split groups
// (SLOTS) have a workgroup for every span, large ones loop.
struct LargeGeom {
    int32_t spans;             // spans per group
    int32_t span_pieces;       // pieces of 8 elements per span; the last span may be shorter
};

constexpr int kLargeUnroll = 4;                          // pieces per lane and step
constexpr int64_t kLargeMinSpanPieces = static_cast<int64_t>(kBlock) * kLargeUnroll;
constexpr int64_t kLargeMaxBlocks = 2048;                // about what is resident at once

// Pieces (of 4 elements in float32, 8 else) per lane and step of a split group's workgroup: 4096
// elements a step, which is the length the host aims a span at.
constexpr int kSplitSpanElements = 4096;
template <int DT> constexpr int kSplitUnroll = kSplitSpanElements / (kBlock * (DT == AQSGD_F32 ? 4 : 8));
constexpr int kSplitMaxSpans = 16;                       // slots read by one wave; a span's codes hold them all

// Their spans are of nearly equal length, so that the last one, too, has codes enough for the
// slots (groups of 32769 elements and more: never fewer than 1800 elements a span).
__host__ __device__ inline LargeGeom split_geometry(const QuantJob& a) {
    LargeGeom g;
    const int spans = (a.group + kSplitSpanElements - 1) / kSplitSpanElements;
    g.spans = spans < kSplitMaxSpans ? spans : kSplitMaxSpans;
    g.span_pieces = (a.cpg + g.spans - 1) / g.spans;
    return g;
}

// Where the spans of a split group leave their maxima for span `span`: one word for each span,
// in the place that span's own codes are going to take (at any byte).
__device__ __forceinline__ u32_any_t* split_slots(const QuantJob& a, const LargeGeom& geom, int i, int64_t g, int span) {
    const int64_t first = static_cast<int64_t>(i) * a.n_per + g * a.group;
    uint8_t* codes_g = a.codes + first * a.bits / 8;
    return reinterpret_cast<u32_any_t*>(codes_g + static_cast<int64_t>(span) * geom.span_pieces * a.bits);
}

// A workgroup's place in its message's rectangle of workgroups.
struct Rect { uint32_t x, y, grid_x, grid_y; };
__device__ __forceinline__ Rect whole_grid() { return {blockIdx.x, blockIdx.y, gridDim.x, gridDim.y}; }

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

template <int DT, bool HAS_BUF, bool SLOTS = false>
__device__ __forceinline__ void large_max_body(const QuantJob& a, const LargeGeom geom, const Rect rect, float* wave_max) {
    constexpr int kUnroll = SLOTS ? kSplitUnroll<DT> : kLargeUnroll;
    constexpr int N = DT == AQSGD_F32 ? 4 : 8;
    constexpr int kEB = ElemBytes<DT>::value;
    const int64_t last_at = a.group - N;
    for (int i = rect.y; SLOTS || i < a.batch; i += rect.grid_y) {
        const int64_t row = a.ids ? sample_id(a.ids, i) : static_cast<int64_t>(i);
        if (large_fresh<HAS_BUF>(a, row)) {
            if constexpr (SLOTS) return;
            else continue;
        }
        const char* src_s = static_cast<const char*>(a.src) + static_cast<int64_t>(i) * a.n_per * kEB;
        const char* m_s = HAS_BUF ? static_cast<const char*>(a.m_buf) + row * a.n_per * kEB : nullptr;
        for (int64_t s = rect.x; SLOTS || s < a.gps * geom.spans; s += rect.grid_x) {
            const int64_t g = s / geom.spans;
            const int64_t e0 = (s - g * geom.spans) * geom.span_pieces * 8;
            const int64_t e1 = min(e0 + static_cast<int64_t>(geom.span_pieces) * 8, static_cast<int64_t>(a.group));
            const char* src_g = src_s + g * a.group * kEB;
            const char* m_g = HAS_BUF ? m_s + g * a.group * kEB : nullptr;
            float mx = 0.0f;
            for (int64_t e = e0 + static_cast<int64_t>(threadIdx.x) * N; e < e1;
                 e += static_cast<int64_t>(kBlock) * N * kUnroll) {
                float x[kUnroll][N], m[kUnroll][N];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) { // past the end: the group's last piece once more
                    const int64_t at = min(e + static_cast<int64_t>(u) * kBlock * N, last_at);
                    load_piece<DT, N>(src_g + at * kEB, x[u]);
                    if constexpr (HAS_BUF) load_piece<DT, N>(m_g + at * kEB, m[u]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
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
            if constexpr (SLOTS) {                       // into every span's slots, see split_slots()
#pragma unroll
                for (int w = 0; w < kBlock / kWave; ++w) mx = __builtin_fmaxf(mx, wave_max[w]);
                const int to = threadIdx.x;
                if (to < geom.spans)
                    split_slots(a, geom, i, g, to)[s - g * geom.spans] = __float_as_uint(mx);
            } else if (threadIdx.x == 0) {
#pragma unroll
                for (int w = 0; w < kBlock / kWave; ++w) mx = __builtin_fmaxf(mx, wave_max[w]);
                atomicMax(reinterpret_cast<unsigned int*>(a.scales) + static_cast<int64_t>(i) * a.gps + g,
                          __float_as_uint(mx));
            }
            if constexpr (SLOTS) break;
        }
        if constexpr (SLOTS) break;
    }
}

template <int DT>
__global__ __launch_bounds__(kBlock)
void large_max_kernel(const QuantJob a, const LargeGeom geom) {
    __shared__ float wave_max[kBlock / kWave];
    if (a.m_buf) large_max_body<DT, true>(a, geom, whole_grid(), wave_max);
    else large_max_body<DT, false>(a, geom, whole_grid(), wave_max);
}

// A group below the 2^-120 floor sends scale 0; one thread rewrites its word while other
// workgroups may still read it, and both values mean "nothing to send" to them.
template <int DT, int BITS, int ROUND, bool HAS_BUF, bool SLOTS = false>
__device__ __forceinline__ void large_quant_body(const QuantJob& a, const LargeGeom geom, const Rect rect) {
    using P = Piece<DT, BITS>;
    constexpr int N = P::elems;
    constexpr int kEB = ElemBytes<DT>::value;
    constexpr int kUnroll = !SLOTS ? kLargeUnroll : DT == AQSGD_F32 && N == 8 ? kSplitUnroll<DT> / 2 : kSplitUnroll<DT>;
    const int64_t last_at = a.group - N;
    for (int i = rect.y; SLOTS || i < a.batch; i += rect.grid_y) {
        const int64_t row = a.ids ? sample_id(a.ids, i) : static_cast<int64_t>(i);
        const int64_t src0 = static_cast<int64_t>(i) * a.n_per;
        const char* src_s = static_cast<const char*>(a.src) + src0 * kEB;
        char* m_s = HAS_BUF ? static_cast<char*>(a.m_buf) + row * a.n_per * kEB : nullptr;
        const bool fresh = large_fresh<HAS_BUF>(a, row);
        if constexpr (HAS_BUF) {
            if (a.seen != nullptr && rect.x == 0 && threadIdx.x == 0) {      // one writer per sample
                a.first[i] = fresh ? 1 : 0;
                if (fresh) a.seen[row] = a.stamp;
            }
        }
        for (int64_t s = rect.x; SLOTS || s < a.gps * geom.spans; s += rect.grid_x) {
            const int64_t g = s / geom.spans;
            const int64_t e0 = (s - g * geom.spans) * geom.span_pieces * 8;
            const int64_t e1 = min(e0 + static_cast<int64_t>(geom.span_pieces) * 8, static_cast<int64_t>(a.group));
            const int64_t goff = g * a.group;
            const char* src_g = src_s + goff * kEB;
            char* m_g = HAS_BUF ? m_s + goff * kEB : nullptr;
            uint8_t* codes_g = a.codes + (src0 + goff) * BITS / 8;
            float* const word = a.scales + static_cast<int64_t>(i) * a.gps + g;
            GroupScale sc;
            if constexpr (SLOTS) {
                if (!fresh) {                            // uniform over the workgroup
                    const int span = static_cast<int>(s - g * geom.spans), from = threadIdx.x % kWave;
                    const uint32_t part = split_slots(a, geom, i, g, span)[min(from, geom.spans - 1)];
                    sc = make_scale<BITS>(team_max<kWave>(__uint_as_float(part)));
                    __syncthreads();                     // every wave has read the slots: codes may go there
                    if (span == 0 && threadIdx.x == 0) *word = sc.s_tx;
                }
            } else if (!fresh) {
                sc = make_scale<BITS>(*word);
                if (e0 == 0 && threadIdx.x == 0 && sc.s_tx == 0.0f) *word = 0.0f;
            }
            for (int64_t e = e0 + static_cast<int64_t>(threadIdx.x) * N; e < e1;
                 e += static_cast<int64_t>(kBlock) * N * kUnroll) {
                float x[kUnroll][N], m[kUnroll][N];
                int64_t at[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    at[u] = min(e + static_cast<int64_t>(u) * kBlock * N, last_at);
                    load_piece<DT, N>(src_g + at[u] * kEB, x[u]);
                    if constexpr (HAS_BUF) load_piece<DT, N>(m_g + at[u] * kEB, m[u]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
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
                        const uint64_t j0 = static_cast<uint64_t>(src0 + goff + at[u]);
                        if (a.group % 4 != 0) {          // uniform over the launch
                            uniforms_any<N>(a.seed, j0, r);
                        } else {                         // whole Philox blocks
#pragma unroll
                            for (int b = 0; b < N; b += 4) block_uniforms(a.seed, (j0 + b) >> 2, &r[b]);
                        }
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
            if constexpr (SLOTS) break;
        }
        if constexpr (SLOTS) break;
    }
}

template <int DT, int BITS, int ROUND>
__device__ __forceinline__ void large_quant_bits(const QuantJob& a, const LargeGeom geom) {
    if (a.m_buf) large_quant_body<DT, BITS, ROUND, true>(a, geom, whole_grid());
    else large_quant_body<DT, BITS, ROUND, false>(a, geom, whole_grid());
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

// ---------------------------------------------------------------------------
// Few wide groups: one workgroup a group leaves most of the chip idle and
// is bound by one compute unit's arithmetic, so each group is split into spans of about 4096
// elements, a workgroup each, in two launches: every span's maximum, then the levels.  The maxima
// travel in the code bytes of the group: each span writes its maximum into a slot of every span,
// and the second launch's workgroup reads its own span's slots before its codes take their place.
// No clearing, no atomics, no memory beyond the call's own, and nothing waits inside a launch.
// (When it pays, and what it measured: split_pays() in the dispatch.)
// ---------------------------------------------------------------------------
template <int DT>
__device__ __forceinline__ void split_max_job(const QuantJob& a, const LargeGeom geom, const Rect rect, float* wave_max) {
    if (a.m_buf) large_max_body<DT, true, true>(a, geom, rect, wave_max);
    else large_max_body<DT, false, true>(a, geom, rect, wave_max);
}

template <int DT>
__global__ __launch_bounds__(kBlock)
void split_max_kernel(AQSGD_QUANT_ARGS, int32_t spans, int32_t span_pieces) {
    __shared__ float wave_max[kBlock / kWave];
    QuantJob a;
    a.src = src; a.ids = ids; a.m_buf = m_buf; a.codes = codes; a.scales = scales;
    a.n_per = n_per; a.gps = gps; a.batch = batch; a.group = group; a.bits = bits;
    a.seen = seen; a.stamp = stamp;
    const LargeGeom geom{spans, span_pieces};
    split_max_job<DT>(a, geom, whole_grid(), wave_max);
}

template <int DT, int BITS, int ROUND>
__device__ __forceinline__ void split_quant_bits(const QuantJob& a, const LargeGeom geom, const Rect rect) {
    if (a.m_buf) large_quant_body<DT, BITS, ROUND, true, true>(a, geom, rect);
    else large_quant_body<DT, BITS, ROUND, false, true>(a, geom, rect);
}

template <int DT, int ROUND>
__device__ __forceinline__ void split_quant_job(const QuantJob& a, const LargeGeom geom, const Rect rect) {
    switch (a.bits) {                                    // uniform over the workgroup
    case 2: split_quant_bits<DT, 2, ROUND>(a, geom, rect); break;
    case 3: split_quant_bits<DT, 3, ROUND>(a, geom, rect); break;
    case 4: split_quant_bits<DT, 4, ROUND>(a, geom, rect); break;
    case 6: split_quant_bits<DT, 6, ROUND>(a, geom, rect); break;
    default: split_quant_bits<DT, 8, ROUND>(a, geom, rect); break;
    }
}

template <int DT, int ROUND>
__global__ __launch_bounds__(kBlock)
void split_quant_kernel(AQSGD_QUANT_ARGS, int32_t spans, int32_t span_pieces) {
    QuantJob a;
    a.src = src; a.ids = ids; a.m_buf = m_buf; a.codes = codes; a.scales = scales;
    a.n_per = n_per; a.gps = gps; a.batch = batch; a.group = group; a.bits = bits;
    a.seed = seed; a.seen = seen; a.first = first; a.stamp = stamp;
    const LargeGeom geom{spans, span_pieces};
    split_quant_job<DT, ROUND>(a, geom, whole_grid());
}

// Per-dtype pieces (defined by AQSGD_INSTANTIATE_ANYGROUP_DTYPE in the dtype's .hip file).
// `through`: float32 without previous messages, groups of whole 16-byte pieces, one step for every workgroup.
template <int DT> hipError_t launch_dequant_odd_dt(bool covers, bool through, const DequantJob& a, hipStream_t stream);
// `parts` workgroups a group, `share` rounds each (1 and all rounds with previous messages).
template <int DT> hipError_t launch_quant_wide_dt(int rounding, int parts, int share, const QuantJob& a, hipStream_t stream);
template <int DT> hipError_t launch_quant_large_dt(int rounding, const QuantJob& a, const LargeGeom& geom,
                                                   hipStream_t stream);
template <int DT> hipError_t launch_quant_split_dt(int rounding, const QuantJob& a, const LargeGeom& geom,
                                                   hipStream_t stream);

// ---- launch tables (instantiated per dtype in aqsgd_anygroup_<dtype>.hip) --------------
template <int DT>
hipError_t launch_dequant_odd_dt(bool covers, bool through, const DequantJob& a, hipStream_t s) {
    if constexpr (DT == AQSGD_F32) {
        if (through) return covers ? launch_dequant_with(dequant_odd_kernel<DT, kOddThrough>, a, s) : hipErrorInvalidValue;
    }
    return covers ? launch_dequant_with(dequant_odd_kernel<DT, kOddOneStep>, a, s)
                  : launch_dequant_with(dequant_odd_kernel<DT, kOddLoops>, a, s);
}

template <int DT>
hipError_t launch_quant_wide_dt(int rounding, int parts, int share, const QuantJob& a, hipStream_t s) {
    auto go = [&](auto kernel) {
        return launch_kernel(kernel, dim3(a.grid_x, a.grid_y, parts), dim3(kWideThreads), s, a.src, a.ids, a.m_buf, a.codes,
                             a.scales, a.group, a.bits | (share << 8), a.n_per, a.gps, a.batch, a.grid_x, a.grid_y,
                             a.stamp, a.seed, a.seen, a.first);
    };
    return rounding == AQSGD_ROUND_STOCHASTIC ? go(quant_wide_kernel<DT, AQSGD_ROUND_STOCHASTIC>)
                                              : go(quant_wide_kernel<DT, AQSGD_ROUND_NEAREST>);
}

template <int DT>
hipError_t launch_quant_large_dt(int rounding, const QuantJob& a, const LargeGeom& geom, hipStream_t s) {
    const int64_t clear_x = (a.gps + kBlock - 1) / kBlock;
    const dim3 grid(a.grid_x, a.grid_y), block(kBlock);
    ProfileSpan span;
    hipError_t err = launch_kernel(large_clear_kernel, dim3(static_cast<unsigned>(clear_x < 1024 ? clear_x : 1024), a.grid_y),
                                   block, s, a);
    if (err == hipSuccess) err = launch_kernel(large_max_kernel<DT>, grid, block, s, a, geom);
    if (err != hipSuccess) return err;
    span.last();
    return rounding == AQSGD_ROUND_STOCHASTIC
               ? launch_kernel(large_quant_kernel<DT, AQSGD_ROUND_STOCHASTIC>, grid, block, s, a, geom)
               : launch_kernel(large_quant_kernel<DT, AQSGD_ROUND_NEAREST>, grid, block, s, a, geom);
}

template <int DT>
hipError_t launch_quant_split_dt(int rounding, const QuantJob& a, const LargeGeom& geom, hipStream_t s) {
    auto go = [&](auto kernel) {
        return launch_kernel(kernel, dim3(a.grid_x, a.grid_y), dim3(kBlock), s, a.src, a.ids, a.m_buf, a.codes,
                             a.scales, a.group, a.bits, a.n_per, a.gps, a.batch, a.grid_x, a.grid_y, a.stamp,
                             a.seed, a.seen, a.first, geom.spans, geom.span_pieces);
    };
    ProfileSpan span;
    const hipError_t err = go(split_max_kernel<DT>);
    if (err != hipSuccess) return err;
    span.last();
    return rounding == AQSGD_ROUND_STOCHASTIC ? go(split_quant_kernel<DT, AQSGD_ROUND_STOCHASTIC>)
                                              : go(split_quant_kernel<DT, AQSGD_ROUND_NEAREST>);
}

#define AQSGD_INSTANTIATE_ANYGROUP_DTYPE(DT)                                                          \
    template hipError_t launch_dequant_odd_dt<DT>(bool, bool, const DequantJob&, hipStream_t);             \
    template hipError_t launch_quant_wide_dt<DT>(int, int, int, const QuantJob&, hipStream_t);             \
    template hipError_t launch_quant_large_dt<DT>(int, const QuantJob&, const LargeGeom&, hipStream_t);   \
    template hipError_t launch_quant_split_dt<DT>(int, const QuantJob&, const LargeGeom&, hipStream_t);

}  // namespace aqsgd
