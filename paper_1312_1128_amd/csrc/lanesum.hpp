// Sums over a wavefront of many per-lane words at once, in registers, by
// recursive halving across the lanes.
#pragma once

#include "common.hpp"

namespace glm {

// Orders this wavefront's LDS accesses around a hand-over between its lanes
// (LDS operations of one wavefront complete in program order).
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The words of one lane handed to the lane that DPP control CTRL names, within
// its 16-lane row.
template <int CTRL>
__device__ inline float row_peer(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// The halving steps inside a row pair lane j with j ^ 8 (row_ror:8), with
// 7 - j inside its 8-lane half (row_half_mirror), then with j ^ 2 and j ^ 1
// (quad_perm); lane bit 3, 2, 1, 0 in turn picks the word kept.
constexpr int kRowStep[4] = {0x128, 0x141, 0x04E, 0x0B1};
constexpr uint64_t kRowHigh[4] = {0xFF00FF00FF00FF00ull, 0xF0F0F0F0F0F0F0F0ull, 0xCCCCCCCCCCCCCCCCull,
                                  0xAAAAAAAAAAAAAAAAull}; // lanes with that bit set

// One halving step inside the rows: the M words of each lane become ceil(M / 2).
// Partner lanes (as step STEP pairs them) keep opposite words of each
// pair (those with the lane bit set: the second) and add the partner's copy; an odd last word is summed
// over both partners, who then hold the same total.
template <int M, int STEP>
__device__ inline void row_halve(float* v)
{
    constexpr int CTRL = kRowStep[STEP];
    constexpr int NP = M / 2;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        float keep, send;
        pick_pair(kRowHigh[STEP], v[2 * p], v[2 * p + 1], keep, send);
        v[p] = keep + row_peer<CTRL>(send);
    }
    if constexpr ((M & 1) != 0) v[NP] = v[M - 1] + row_peer<CTRL>(v[M - 1]);
}

// Totals over the wavefront of NA per-lane words (NA even), by recursive
// halving across the lanes, in registers.  The 32-lane halves swap the half of
// the words that the other one keeps (v_permlane32_swap: lane i < 32 exchanges
// its second operand with the first operand of lane i + 32) and add, so that
// half h holds words h H .. h H + H - 1 (H = NA / 2), each summed over two
// lanes; the two 16-lane rows of each half do the same with v_permlane16_swap,
// so that row R = 2 h + r holds words h H + r Q .. h H + r Q + Q - 1
// (Q = ceil(H / 2), a zero word filling an odd H) summed over four lanes; four
// halving steps inside the rows complete the sums over each row's 16 lanes.
// A lane's total is that of the word word_slot names.  Every lane of the
// wavefront takes part.
template <int NA>
__device__ inline float word_totals(const float* a)
{
    static_assert(NA % 2 == 0 && NA <= 64, "an even number of words");
    constexpr int H = NA / 2;
    constexpr int Q = (H + 1) / 2;
    constexpr int M2 = (Q + 1) / 2, M3 = (M2 + 1) / 2, M4 = (M3 + 1) / 2;
    static_assert((M4 + 1) / 2 == 1, "one word per lane after four steps");
    float b[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[k]), __float_as_uint(a[H + k]), false,
                                                        false);
        b[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    float c[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const float hi = k + Q < H ? b[k + Q] : 0.0f;
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(b[k]), __float_as_uint(hi), false, false);
        c[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    row_halve<Q, 0>(c);
    row_halve<M2, 1>(c);
    row_halve<M3, 2>(c);
    row_halve<M4, 3>(c);
    return c[0];
}

// The word whose total word_totals leaves in this lane: the same halving
// steps applied to word indices.  -1 where the lane holds no word, or a copy of
// a total that another lane holds too (only one lane adds it).
template <int NA>
__device__ inline int word_slot(int lane)
{
    constexpr int H = NA / 2;
    constexpr int Q = (H + 1) / 2;
    const int j = lane & 15, R = lane >> 4;
    int wd[Q];
    bool own[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        wd[k] = k;
        own[k] = true;
    }
    int m = Q;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const bool hi = ((j >> (3 - st)) & 1) != 0;
        const int np = m / 2;
#pragma unroll
        for (int p = 0; p < Q / 2; ++p) {
            if (p < np) {
                wd[p] = hi ? wd[2 * p + 1] : wd[2 * p];
                own[p] = hi ? own[2 * p + 1] : own[2 * p];
            }
        }
        if (m & 1) {
            wd[np] = wd[m - 1];
            own[np] = own[m - 1] && !hi;
        }
        m = np + (m & 1);
    }
    const int i = (R & 1) * Q + wd[0];
    return own[0] && i < H ? (R >> 1) * H + i : -1;
}

// The same in FP64 (two dwords per exchange): totals of FP32 words whose sum
// over the lanes is taken in FP64.
__device__ inline double lane_pair(uint32_t lo, uint32_t hi) { return __hiloint2double((int)hi, (int)lo); }

template <int CTRL>
__device__ inline double row_peer64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

template <int M, int STEP>
__device__ inline void row_halve64(double* v)
{
    constexpr int CTRL = kRowStep[STEP];
    constexpr int NP = M / 2;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        double keep, send;
        pick_pair(kRowHigh[STEP], v[2 * p], v[2 * p + 1], keep, send);
        v[p] = keep + row_peer64<CTRL>(send);
    }
    if constexpr ((M & 1) != 0) v[NP] = v[M - 1] + row_peer64<CTRL>(v[M - 1]);
}

template <int NA>
__device__ inline double word_totals64(const float* a)
{
    static_assert(NA % 2 == 0 && NA <= 64, "an even number of words");
    constexpr int H = NA / 2;
    constexpr int Q = (H + 1) / 2;
    constexpr int M2 = (Q + 1) / 2, M3 = (M2 + 1) / 2, M4 = (M3 + 1) / 2;
    static_assert((M4 + 1) / 2 == 1, "one word per lane after four steps");
    double b[H];
#pragma unroll
    for (int k = 0; k < H; ++k) { // FP32 words: one exchange moves a whole word
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[k]), __float_as_uint(a[H + k]), false,
                                                        false);
        b[k] = (double)__uint_as_float(r[0]) + (double)__uint_as_float(r[1]);
    }
    double c[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const double hi = k + Q < H ? b[k + Q] : 0.0;
        const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(b[k]), (uint32_t)__double2loint(hi),
                                                        false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(b[k]), (uint32_t)__double2hiint(hi),
                                                        false, false);
        c[k] = lane_pair(l[0], h[0]) + lane_pair(l[1], h[1]);
    }
    row_halve64<Q, 0>(c);
    row_halve64<M2, 1>(c);
    row_halve64<M3, 2>(c);
    row_halve64<M4, 3>(c);
    return c[0];
}

// Totals over the wavefront of four FP64 words: row R (lanes 16 R .. 16 R + 15)
// ends with word R's.
__device__ inline double row_word4(const double* a)
{
    double b[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) { // half h of the wavefront keeps words 2 h, 2 h + 1
        const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)__double2loint(a[k]), (uint32_t)__double2loint(a[2 + k]),
                                                        false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)__double2hiint(a[k]), (uint32_t)__double2hiint(a[2 + k]),
                                                        false, false);
        b[k] = lane_pair(l[0], h[0]) + lane_pair(l[1], h[1]);
    }
    const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(b[0]), (uint32_t)__double2loint(b[1]), false,
                                                    false);
    const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(b[0]), (uint32_t)__double2hiint(b[1]), false,
                                                    false);
    double v = lane_pair(l[0], h[0]) + lane_pair(l[1], h[1]);
    v += row_peer64<kRowStep[0]>(v);
    v += row_peer64<kRowStep[1]>(v);
    v += row_peer64<kRowStep[2]>(v);
    return v + row_peer64<kRowStep[3]>(v);
}

// Smallest, largest value and sum over the wavefront, in every lane (butterfly
// exchanges in registers: pairs 32, 16, 8, 4, 2, 1 lanes apart).
template <class Op>
__device__ inline double wave_all(double v, Op op)
{
    auto l = __builtin_amdgcn_permlane32_swap((uint32_t)__double2loint(v), (uint32_t)__double2loint(v), false, false);
    auto h = __builtin_amdgcn_permlane32_swap((uint32_t)__double2hiint(v), (uint32_t)__double2hiint(v), false, false);
    v = op(lane_pair(l[0], h[0]), lane_pair(l[1], h[1]));
    l = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(v), (uint32_t)__double2loint(v), false, false);
    h = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(v), (uint32_t)__double2hiint(v), false, false);
    v = op(lane_pair(l[0], h[0]), lane_pair(l[1], h[1]));
    v = op(v, row_peer64<kRowStep[0]>(v));
    v = op(v, row_peer64<kRowStep[1]>(v));
    v = op(v, row_peer64<kRowStep[2]>(v));
    return op(v, row_peer64<kRowStep[3]>(v));
}
__device__ inline double wave_min(double v)
{
    return wave_all(v, [](double a, double b) { return fmin(a, b); });
}
__device__ inline double wave_max(double v)
{
    return wave_all(v, [](double a, double b) { return fmax(a, b); });
}
__device__ inline double wave_sum(double v)
{
    return wave_all(v, [](double a, double b) { return a + b; });
}

} // namespace glm
