// Pieces of the routing that more than one translation unit uses.
#pragma once
#include "kernels.hpp"

namespace lexi {

// ---------------------------------------------------------------------------------------------------------
// write_work_list: the expert table and the tiles of the two grouped GEMMs, by one wave (lane = expert, `total` = its
// rows); returns the expert's first permuted row.
// ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ int32_t write_work_list(int32_t total, int E, const WorkPlan& plan, int32_t* __restrict__ counts,
                                                   int32_t* __restrict__ offsets, int32_t* __restrict__ sched) {
    const int lane = threadIdx.x & 63;
    const int32_t off = wave_inclusive_sum(total) - total;
    if (lane < E) {
        counts[lane] = total;
        offsets[lane] = off;
    }
    if (lane == 63) offsets[E] = off + total;       // lanes >= E hold no rows
    sched[kSchedOff + lane] = off;
    sched[kSchedCount + lane] = total;
#pragma unroll
    for (int g = 0; g < 2; ++g)
        sched[kSchedTiles + 64 * g + lane] = wave_inclusive_sum((total + plan.tile_rows[g] - 1) / plan.tile_rows[g]);
    return off;
}

// The top-k of TM tokens by one wave (lane = expert): total[m] are the logits before the bias; lane e learns whether token m took
// expert e, lane s < k the expert and the logit of slot s.  k rounds of {wave maximum by DPP, ballot of the lanes that hold it, lowest
// set bit}: the lowest index among equal logits wins; comparisons are on floats, so +0 == -0.
// Inputs are finite by contract.  A NaN logit (one NaN or Inf activation is enough) compares unequal to every maximum, which would
// leave the ballot empty and the expert index undefined; it ranks as -inf instead, so every round selects a valid expert (all-NaN
// row: experts 0..k-1) and the token's gates and output come out NaN.
template <int TM>
__device__ __forceinline__ void pick_experts(float (&total)[TM], const float* __restrict__ bias, int E, int k, bool (&taken)[TM],
                                             int32_t (&sel)[TM], float (&val)[TM]) {
    const int lane = threadIdx.x & 63;
    const bool lane_valid = lane < E;
    const float b = (bias != nullptr && lane_valid) ? bias[lane] : 0.0f;
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        if (bias != nullptr) total[m] = total[m] + b;
        total[m] = total[m] == total[m] ? total[m] : -INFINITY;
        taken[m] = false; sel[m] = 0; val[m] = -INFINITY;
    }
    for (int s = 0; s < k; ++s) {
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            const bool open = lane_valid && !taken[m];
            const float mx = wave_max(open ? total[m] : -INFINITY);
            const int e_star = __builtin_ctzll(__ballot(open && total[m] == mx));   // lowest index among equal logits
            if (lane == e_star) taken[m] = true;
            if (lane == s) { sel[m] = e_star; val[m] = mx; }
        }
    }
}
// Softmax over the selected: lane s < k gets the gate of slot s.
__device__ __forceinline__ float gate_of(float val, int k) {
    const float v0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(val), 0));   // slot 0 holds the largest
    const float ex = (int)(threadIdx.x & 63) < k ? __expf(val - v0) : 0.0f;
    return ex / wave_sum(ex);
}

// ---------------------------------------------------------------------------------------------------------
// Selection of a few tokens by every workgroup of a launch for itself (T <= MAXT <= kSelectMaxT): the experts token t selects as bits
// of s_mask[t].  Logits are the ordered sums of the segment partials (plus bias), the selection the total order (logit
// descending, index ascending), as everywhere.  A wave takes tokens wave, wave + NW, ...; `picked` is called for
// each of them with the token, and per lane s < k the expert and the logit of slot s.
// All segments' partials of a token (up to 16 at a time) are requested together: one round trip.
// ---------------------------------------------------------------------------------------------------------
template <int NW, int MAXT, typename Picked>
__device__ __forceinline__ void select_tokens(const float* __restrict__ partial, const float* __restrict__ bias, int T, int nseg,
                                              int E, int k, uint64_t* s_mask, Picked picked) {
    constexpr int TM = MAXT / NW;                // tokens per wave, interleaved
    static_assert(TM * NW == MAXT, "");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= T) return;
    float total[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) total[m] = 0.0f;
    for (int s0 = 0; s0 < nseg; s0 += 16) {
        float p[16][TM];
#pragma unroll
        for (int c = 0; c < 16; ++c)
#pragma unroll
            for (int m = 0; m < TM; ++m)         // (past the last segment and token: the last one again, unused)
                p[c][m] = partial[((size_t)min(s0 + c, nseg - 1) * T + min(wave + m * NW, T - 1)) * 64 + lane];
#pragma unroll
        for (int c = 0; c < 16; ++c)
            if (s0 + c < nseg) {
#pragma unroll
                for (int m = 0; m < TM; ++m) total[m] = s0 + c == 0 ? p[c][m] : total[m] + p[c][m];
            }
    }
    bool taken[TM];
    int32_t sel[TM];
    float val[TM];
    pick_experts<TM>(total, bias, E, k, taken, sel, val);
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        const int t = wave + m * NW;
        if (t >= T) break;
        const uint64_t mask = __ballot(taken[m]);
        if (lane == 0) s_mask[t] = mask;
        picked(t, sel[m], val[m]);
    }
}

}  // namespace lexi
