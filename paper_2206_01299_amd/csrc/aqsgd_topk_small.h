// Sparsified backward message, many groups of at most 512 entries: several groups to a wave.
//
// A team of 4, 8 or 16 lanes owns a group, one to four chunks of eight entries per lane, so a wave
// takes 64 / TEAM consecutive groups at once.  The sender is bound by the number of vector
// instructions, and the wave-per-group kernels (aqsgd_topk.h) spend them, two to four histograms in
// LDS with a scan over the wave each among them, on lanes without entries.  Here the threshold is
// found by bisection on the magnitudes' bit patterns: a step counts the entries below a pattern, ten
// instructions for a lane's eight entries (packed 16-bit differences, whose sign bits a byte permute
// spreads over bytes for a population count) and two to four for the sum over the team, and all
// teams of the wave share the steps.  They look at the eight octaves below a group's largest entry,
// ten to fifteen bits, and end where the count is exact in every team.
//
// A group's `keep` bytes follow the previous group's, so the bytes of a wave are one string, which
// leaves as 4-byte stores.
//
// Measured, a wave per group -> here, us a launch: sender, 65536 groups of 64, a fifth kept, float16
// 34.2 -> 9.4, binary32 48.3 -> 9.8; of 256, 35.5 -> 22.6 and 52.1 -> 23.9; receiver, of 64, 19.1 ->
// 4.8 and 18.0 -> 6.8 (8.4 and 16.8 MB written).  The floor of the sender of 256 in binary32 is its
// 67 MB, 12.5 us: levels, staging and the search are what it spends the rest on.
#pragma once

#include "aqsgd_topk.h"

namespace aqsgd {

// Patterns of a lane's entries, CPL chunks of eight.  16-bit types hold the magnitudes in pairs;
// of binary32 the magnitudes are formed again from the entries where they are needed.
template <int DT>
__device__ __forceinline__ uint32_t magnitude_word(const Raw<DT>& r, int e) {
    static_assert(DT == AQSGD_F32, "one entry a word");
    return __float_as_uint(e < 4 ? r.lo[e & 3] : r.hi[e & 3]) & 0x7fffffffu;
}

// The sign bits of eight packed 16-bit values, a byte of ones or zeros for each (a selector of
// 8 to 11 makes v_perm_b32 repeat the sign of one of its four halves): entries 0-3 and 4-7.
struct SignBytes { uint32_t lo, hi; };
__device__ __forceinline__ SignBytes sign_bytes16(const uint32_t (&d)[4]) {
    return {__builtin_amdgcn_perm(d[1], d[0], 0x0b0a0908u), __builtin_amdgcn_perm(d[3], d[2], 0x0b0a0908u)};
}
// ... as a bit for each, entry e at bit e.
__device__ __forceinline__ uint32_t bits_of_bytes(const SignBytes& b) {
    return __builtin_amdgcn_sad_u8((b.lo & 0x08040201u) | (b.hi & 0x80402010u), 0u, 0u);
}

// Number of a lane's entries whose packed pattern is below `t` (all of them below 2^15).
template <int CPL>
__device__ __forceinline__ uint32_t below_pairs(const uint32_t (&pair)[CPL][4], uint32_t t) {
    const uint32_t tt = t | (t << 16);
    uint32_t n = 0;
#pragma unroll
    for (int k = 0; k < CPL; k += 4) {                   // four chunks' sign bytes fill a word's bits
        uint32_t bits = 0;
#pragma unroll
        for (int j = 0; j < 4 && k + j < CPL; ++j) {
            uint32_t d[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i] = pk_sub_u16(pair[k + j][i], tt);
            const SignBytes s = sign_bytes16(d);
            bits |= (s.lo & (0x01010101u << (2 * j))) | (s.hi & (0x02020202u << (2 * j)));
        }
        n += static_cast<uint32_t>(__builtin_popcount(bits));
    }
    return n;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_add_step(uint32_t v) {
    return v + static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xf, 0xf, true));
}

// Sum over the team, in every lane of it (the exchanges of team_max).
template <int TEAM>
__device__ __forceinline__ uint32_t team_sum(uint32_t v) {
    static_assert(TEAM <= 16, "a team lies in one row of 16 lanes");
    if constexpr (TEAM >= 2) v = dpp_add_step<0xB1>(v);      // quad_perm [1,0,3,2]
    if constexpr (TEAM >= 4) v = dpp_add_step<0x4E>(v);      // quad_perm [2,3,0,1]
    if constexpr (TEAM >= 8) v = dpp_add_step<0x141>(v);     // row_half_mirror
    if constexpr (TEAM >= 16) v = dpp_add_step<0x140>(v);    // row_mirror
    return v;
}

// Exclusive prefix sum over the lanes of the team.
template <int TEAM>
__device__ __forceinline__ uint32_t team_exclusive_sum(uint32_t x, int lane) {
    uint32_t total;
    const uint32_t before = wave_inclusive_sum(x, lane, total) - x;
    return before - static_cast<uint32_t>(__shfl(static_cast<int>(before), lane & ~(TEAM - 1), kWave));
}

// For every chunk row of the lane's counts (each below 2^16 over the team): the sum of what comes
// before the lane's chunk in entry order, rows before and lanes before in its row.
template <int TEAM, int CPL>
__device__ __forceinline__ void before_in_team(const uint32_t (&cnt)[CPL], int lane, uint32_t (&before)[CPL]) {
    uint32_t row = 0;
#pragma unroll
    for (int k = 0; k < CPL; k += 2) {
        const uint32_t second = k + 1 < CPL ? cnt[k + 1 < CPL ? k + 1 : k] : 0u;
        const uint32_t packed = cnt[k] | (second << 16);
        const uint32_t x = team_exclusive_sum<TEAM>(packed, lane);
        before[k] = row + (x & 0xffffu);
        if (k + 1 < CPL || k + 2 < CPL) {
            const uint32_t total = team_sum<TEAM>(packed);
            row += total & 0xffffu;
            if (k + 1 < CPL) before[k + 1 < CPL ? k + 1 : k] = row + (x >> 16);
            row += total >> 16;
        }
    }
}

// What the bisection works on: 15-bit keys that keep the order of the magnitudes over the eight
// octaves below the group's largest (`top`) and are 0 below.  key = (pattern - base) >> shift.
template <int DT> struct SmallKey;
template <> struct SmallKey<AQSGD_F16>  { static constexpr int bits = 13, shift = 0; };
template <> struct SmallKey<AQSGD_BF16> { static constexpr int bits = 10, shift = 0; };
template <> struct SmallKey<AQSGD_F32>  { static constexpr int bits = 15, shift = 11; };

__device__ __forceinline__ uint32_t pk_sub_sat_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2_t, a),
                                                                      __builtin_bit_cast(u16x2_t, b)));
}

// The largest pattern t with at most `drop` = group - keep entries below it, which is the keep-th
// largest one, or any pattern with exactly `drop` entries below it.  Returns it with the number
// of entries below.  Lanes without entries (`valid` false) count nothing.
template <int DT, int TEAM, int CPL>
__device__ __forceinline__ void small_threshold(const Raw<DT> (&raw)[CPL], const bool (&valid)[CPL], uint32_t top,
                                                uint32_t drop, uint32_t& t, uint32_t& below) {
    using Key = SmallKey<DT>;
    constexpr uint32_t kSpan = (1u << (Key::bits + Key::shift)) - 1;
    const uint32_t base = top > kSpan ? top - kSpan : 0u;
    uint32_t pair[CPL][4];
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        if constexpr (DT == AQSGD_F32) {
            uint32_t v[kChunk];
#pragma unroll
            for (int e = 0; e < kChunk; ++e)
                v[e] = __builtin_elementwise_sub_sat(magnitude_word<DT>(raw[k], e), base) << (16 - Key::shift);
#pragma unroll
            for (int i = 0; i < 4; ++i) pair[k][i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], 0x07060302u);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) pair[k][i] = pk_sub_sat_u16(raw[k].v[i] & 0x7fff7fffu, base | (base << 16));
        }
        if (!valid[k]) {
#pragma unroll
            for (int i = 0; i < 4; ++i) pair[k][i] = 0x7fff7fffu;    // not below any key
        }
    }
    // ---- the key's bits from the highest that any group of the wave has ------------------------
    uint32_t key = 0, key_below = 0;
    uint32_t bit = 1u << (Key::bits - 1);
    const uint32_t top_key = (top - base) >> Key::shift;
    while (bit > 1 && __ballot(top_key >= bit) == 0) bit >>= 1;
    for (; bit != 0 && __ballot(key_below != drop) != 0; bit >>= 1) {      // wave-uniform
        const uint32_t n = team_sum<TEAM>(below_pairs<CPL>(pair, key + bit));
        const bool enough = n <= drop;
        key = enough ? key + bit : key;
        key_below = enough ? n : key_below;
    }
    // ---- where that was not enough: equal keys of different patterns, a threshold more than eight
    //      octaves below the largest.  At most `drop` entries are below lo, more below hi. ---------
    uint32_t lo = key == 0 ? 0u : base + (key << Key::shift);
    uint32_t hi = base + ((key + 1) << Key::shift);
    while (__ballot(key_below != drop && hi - lo > 1) != 0) {        // wave-uniform; halves hi - lo of such teams
        const uint32_t mid = (lo + hi) >> 1;
        uint32_t n = 0;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
#pragma unroll
            for (int e = 0; e < kChunk; ++e) {
                uint32_t u;
                if constexpr (DT == AQSGD_F32) u = magnitude_word<DT>(raw[k], e);
                else u = (e % 2 ? raw[k].v[e / 2] >> 16 : raw[k].v[e / 2]) & 0x7fffu;
                n += valid[k] && u < mid ? 1u : 0u;
            }
        }
        n = team_sum<TEAM>(n);
        const bool enough = n <= drop;
        lo = enough ? mid : lo;
        hi = enough ? hi : mid;
        key_below = enough ? n : key_below;
    }
    t = lo;
    below = key_below;
}

// Bit e of the result: entry e's magnitude is below t (OR_EQUAL: or equal to it).
template <int DT, bool OR_EQUAL>
__device__ __forceinline__ uint32_t below_mask(const Raw<DT>& r, uint32_t t) {
    if constexpr (DT == AQSGD_F32) {
        uint32_t m = 0;
#pragma unroll
        for (int e = kChunk - 1; e >= 0; --e) {          // patterns below 2^31: the sign of a difference, last entry first
            const uint32_t u = magnitude_word<DT>(r, e);
            m = __builtin_amdgcn_alignbit(m, OR_EQUAL ? ~(t - u) : u - t, 31);
        }
        return m & 0xffu;
    } else {
        const uint32_t tt = t | (t << 16);
        uint32_t d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t u = r.v[i] & 0x7fff7fffu;
            d[i] = OR_EQUAL ? ~pk_sub_u16(tt, u) : pk_sub_u16(u, tt);
        }
        return bits_of_bytes(sign_bytes16(d));
    }
}

template <int DT, int TEAM, int CPL, int ROUND>
__device__ __forceinline__ void topk_small_quant(const TopkArgs& a, int64_t g0, int live, const uint32_t (&cc)[CPL],
                                                 const bool (&valid)[CPL], int lane, uint8_t* stage) {
    constexpr int kEB = ElemBytes<DT>::value;
    constexpr int kSpare = kWave * CPL * kChunk;         // staging bytes of the wave; behind them one a lane to spare
    const int team = lane / TEAM;
    // a team past the last group reads that group again; nothing of it counts or is stored
    const int64_t g = g0 + min(team, live - 1);
    const int64_t e0 = g * a.group;
    Raw<DT> raw[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) raw[k] = load_raw_at<DT>(static_cast<const char*>(a.grad) + (e0 + cc[k] * kChunk) * kEB);
    __builtin_amdgcn_sched_barrier(0);

    // ---- the group's largest magnitude, and the keep-th largest --------------------------------
    uint32_t top = 0;                                    // a lane past the group repeats its last chunk: harmless here
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        if constexpr (DT == AQSGD_F32) {
#pragma unroll
            for (int e = 0; e < kChunk; ++e) top = max(top, magnitude_word<DT>(raw[k], e));
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) top = pk_max_u16(top, raw[k].v[i] & 0x7fff7fffu);
        }
    }
    if constexpr (DT != AQSGD_F32) top = max(top & 0xffffu, top >> 16);
    top = __float_as_uint(team_max<TEAM>(__uint_as_float(top)));     // an integer maximum over the lanes
    GroupScale sc;
    if constexpr (DT == AQSGD_F32) sc = make_scale<kTopkBits>(__uint_as_float(top));
    else sc = make_scale<kTopkBits>(f32_of_bits16<DT>(top));
    const uint32_t drop = static_cast<uint32_t>(a.group - a.keep);
    uint32_t t, below;
    small_threshold<DT, TEAM, CPL>(raw, valid, top, drop, t, below);

    // ---- keep flags: everything from the threshold up, but of those equal to it only the first ----
    uint32_t keepb[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) keepb[k] = valid[k] ? ~below_mask<DT, false>(raw[k], t) & 0xffu : 0u;
    if (__ballot(below != drop) != 0) {                  // some team has equals to choose from (wave-uniform)
        uint32_t equal[CPL], ties[CPL], ties_before[CPL], ties_mine = 0;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            equal[k] = keepb[k] & below_mask<DT, true>(raw[k], t);
            ties[k] = static_cast<uint32_t>(__builtin_popcount(equal[k]));
            ties_mine += ties[k];
        }
        const int equal_kept = static_cast<int>(team_sum<TEAM>(ties_mine) - (drop - below));
        before_in_team<TEAM, CPL>(ties, lane, ties_before);
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const int allowed = equal_kept - static_cast<int>(ties_before[k]);
            keepb[k] = (keepb[k] & ~equal[k]) | (static_cast<int>(ties[k]) <= allowed ? equal[k] : 0u);
            if (allowed > 0 && allowed < static_cast<int>(ties[k])) {            // the cut falls inside this chunk
                int seen = 0;
#pragma unroll
                for (int e = 0; e < kChunk; ++e) {
                    const uint32_t eq = (equal[k] >> e) & 1u;
                    if (eq && seen < allowed) keepb[k] |= 1u << e;
                    seen += static_cast<int>(eq);
                }
            }
        }
    }

    // ---- levels of the kept entries into the wave's string ---------------------------------------
    const bool stores = team < live;
    uint32_t kept[CPL], before[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) kept[k] = static_cast<uint32_t>(__builtin_popcount(keepb[k]));
    before_in_team<TEAM, CPL>(kept, lane, before);
    const int spare = kSpare + lane;                     // where an entry that is not kept goes
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        float f[kChunk], r[kChunk];
        if constexpr (ROUND == AQSGD_ROUND_STOCHASTIC) {
            chunk_uniforms(a.seed, static_cast<uint64_t>(e0) + cc[k] * kChunk, r);
        } else {
#pragma unroll
            for (int e = 0; e < kChunk; ++e) r[e] = kNearestOffset32;
        }
        unpack_raw<DT>(raw[k], f);
        int ahead = team * a.keep + static_cast<int>(before[k]) - spare;         // a team that stores nothing: past the string
#pragma unroll
        for (int e = 0; e < kChunk; ++e) {
            const int on = static_cast<int>((keepb[k] >> e) & 1u);
            const float q = level_of<kTopkBits, ROUND>(f[e], sc, r[e]);
            stage[__mul24(on, ahead) + spare] = static_cast<uint8_t>(__builtin_amdgcn_cvt_pk_u8_f32(q, 0, 0));
            ahead += on;
        }
        if (valid[k] && stores) a.bitmap[e0 / kChunk + cc[k]] = static_cast<uint8_t>(keepb[k]);
    }
    if (lane % TEAM == 0 && stores) a.scales[g] = sc.s_tx;
    wave_lds_sync();
    string_out(a.codes + g0 * a.keep, stage, live * a.keep, lane);
    wave_lds_sync();                                     // the next groups reuse the staging bytes
}

template <int DT, int TEAM, int CPL>
__device__ __forceinline__ void topk_small_dequant(const TopkArgs& a, int64_t g0, int live, const uint32_t (&cc)[CPL],
                                                   const bool (&valid)[CPL], int lane, uint8_t* stage) {
    constexpr int kEB = ElemBytes<DT>::value;
    const int team = min(lane / TEAM, live - 1);
    const bool stores = lane / TEAM < live;
    const int64_t g = g0 + team;
    const int64_t e0 = g * a.group;
    uint32_t bm[CPL], kept[CPL], before[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) bm[k] = a.bitmap[e0 / kChunk + cc[k]];
    const float s_tx = a.scales[g];
    string_in(stage, a.codes + g0 * a.keep, live * a.keep, lane);
    wave_lds_sync();
    const GroupScale sc = scale_from_wire<kTopkBits>(s_tx);
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        if (!valid[k]) bm[k] = 0;
        kept[k] = static_cast<uint32_t>(__builtin_popcount(bm[k]));
    }
    before_in_team<TEAM, CPL>(kept, lane, before);
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        // at most team * keep + group: inside the staging bytes also for a bitmap that disagrees with `keep`
        uint32_t pos = static_cast<uint32_t>(team * a.keep) + before[k];
        float x[kChunk];
#pragma unroll
        for (int e = 0; e < kChunk; ++e) {
            const uint32_t on = (bm[k] >> e) & 1u;
            const float v = value_of(static_cast<float>(stage[pos]), sc);
            x[e] = on ? v : 0.0f;
            pos += on;
        }
        // written through at every size: streaming, in us, float16 512 groups of 64 2.07 -> 2.17, bfloat16 131072
        // groups of 64 6.28 -> 6.50, float16 262144 of 128 14.9 -> 15.4
        if (valid[k] && stores)
            store_raw_at<DT>(static_cast<char*>(a.out) + (e0 + cc[k] * kChunk) * kEB, pack_raw<DT>(x), true);
    }
    wave_lds_sync();
}

// MODE and the arguments as topk_kernel's; one wave a workgroup.
template <int DT, int TEAM, int CPL, int MODE>
__global__ __launch_bounds__(kTopkBlock)
void topk_small_kernel(void* data, uint8_t* bitmap, uint8_t* codes, float* scales, int64_t n_groups, int32_t group,
                       int32_t cpg, int32_t keep, uint32_t n_blocks, uint64_t seed) {
    TopkArgs a;
    a.grad = data; a.out = data; a.bitmap = bitmap; a.codes = codes; a.scales = scales;
    a.n_groups = n_groups; a.group = group; a.cpg = cpg; a.keep = keep; a.stochastic = MODE == 2; a.seed = seed;
    constexpr int kTeams = kWave / TEAM;
    __shared__ __align__(16) uint8_t stage[kWave * CPL * kChunk + kWave];
    const int lane = threadIdx.x;
    bool valid[CPL];
    uint32_t cc[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        const int c = k * TEAM + lane % TEAM;
        valid[k] = c < cpg;
        cc[k] = static_cast<uint32_t>(min(c, cpg - 1));
    }
    for (int64_t g0 = static_cast<int64_t>(xcd_contiguous_slot(blockIdx.x, n_blocks)) * kTeams; g0 < n_groups;
         g0 += static_cast<int64_t>(n_blocks) * kTeams) {
        const int live = static_cast<int>(min(n_groups - g0, static_cast<int64_t>(kTeams)));
        if constexpr (MODE == 0) topk_small_dequant<DT, TEAM, CPL>(a, g0, live, cc, valid, lane, stage);
        else if constexpr (MODE == 1) topk_small_quant<DT, TEAM, CPL, AQSGD_ROUND_NEAREST>(a, g0, live, cc, valid, lane, stage);
        else topk_small_quant<DT, TEAM, CPL, AQSGD_ROUND_STOCHASTIC>(a, g0, live, cc, valid, lane, stage);
    }
}

// Lanes of a team and chunks a lane, or lanes = 0: one wave per group (aqsgd_topk.h).  That kernel's
// waves hide each other's waiting until there are two or three of them on each of the chip's 1024
// SIMDs, and a launch with fewer groups is over sooner with short waves, one group each; from there
// on its time grows with the groups.  Measured, sender in us, wave per group -> teams, float16 and
// binary32 below each line and above it:
//   cpg  4, from  2048 groups: 1024 3.31 -> 3.53, 3.80 -> 3.75;  2048 3.69 -> 3.58, 4.36 -> 3.75
//   cpg 16, from  3072 groups: 2048 3.74 -> 3.84, 4.41 -> 4.34;  4096 4.63 -> 3.90, 6.02 -> 4.75
//   two chunks a lane, from 24576: 16384 6.29 -> 5.99, 6.87 -> 7.21;  65536 14.8 -> 13.1, 15.5 -> 13.8
//   cpg 32, from  6144 groups: 4096 4.80 -> 5.12, 6.00 -> 6.37;  8192 7.10 -> 6.07, 10.0 -> 7.46
//   cpg 64, from 16384 groups, binary32: 8192 10.9 -> 11.7;  16384 17.9 -> 15.9;  65536 59 -> 41
//     (float16 stays: 16384 11.7 -> 12.8, 65536 37.6 -> 36.3)
// and the receivers (which have no search):
//   cpg up to 16 at every size: 64 groups of 32 2.32 -> 2.32, 1024 of 88 2.83 -> 2.42
//   cpg 32, from 2048 groups: 1024 2.46 -> 2.65, 2.61 -> 2.73;  2048 2.90 -> 2.74, 2.96 -> 2.94
//   cpg 64, from 8192 groups, 16 bits: 4096 3.43 -> 3.7;  8192 4.52 -> 3.99 (binary32 6.53 -> 6.80)
struct TopkSmallShape { int lanes, cpl; };
inline TopkSmallShape topk_small_shape(int dtype, bool sender, int cpg, int64_t n_groups) {
    const TopkSmallShape wave{0, 0};
    if (cpg <= 8) return sender && n_groups < 2048 ? wave : TopkSmallShape{cpg <= 4 ? 4 : 8, 1};
    if (cpg <= 16) return sender && n_groups < 3072 ? wave : n_groups < 24576 ? TopkSmallShape{16, 1} : TopkSmallShape{8, 2};
    if (cpg <= 32) return n_groups < (sender ? 6144 : 2048) ? wave : TopkSmallShape{16, 2};
    if (cpg <= 64 && sender == (dtype == AQSGD_F32)) return n_groups < (sender ? 16384 : 8192) ? wave : TopkSmallShape{16, 4};
    return wave;
}

hipError_t launch_topk_small(int dtype, TopkSmallShape shape, bool sender, unsigned blocks, const TopkArgs& a, hipStream_t stream);

}  // namespace aqsgd
