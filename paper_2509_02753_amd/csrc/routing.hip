// Routing kernels: fp32 router GEMM + wave-level top-k + softmax over the selected, and the deterministic
// token-to-expert permutation (per-block histogram -> scan -> scatter).
//
// Paper Sec. 2: G(x) = Softmax(TopK[x * W_g]); k is a launch argument (Algorithm 1's UpdateTopk).
#include "routing_common.hpp"
#include <utility>

namespace lexi {

// ---------------------------------------------------------------------------------------------------------
// The fp32 logit of (token t, expert e) has ONE defined evaluation order: d is cut into segments of 128; inside a
// segment the partial starts at +0 and takes one fused multiply-add per element, ascending; the partials are added
// in ascending segment order; the bias is added last.  The segment partials are independent chains, which is where
// the parallelism comes from: one wave computes one segment.
// ---------------------------------------------------------------------------------------------------------

// router_partial_small_kernel (T <= kSmallRouterMaxT): one wave = one segment of one token, lane = expert.  The segment's
// 128 router weights of the lane's expert sit in registers (128 coalesced loads in flight at once), the token's x values
// are wave-uniform (scalar loads): one 128-long chain of fused multiply-adds, partials to partial[seg][t][e].  A few
// tokens are bound by latency: d/128 * T workgroups each pull 32 KB of W, where one workgroup per token block would pull
// all of it through one CU.
template <bool IS_BF16>
__global__ void __launch_bounds__(64)
router_partial_small_kernel(const void* __restrict__ x, const float* __restrict__ w_router, int T, int d, int E,
                            float* __restrict__ partial) {
    const int lane = threadIdx.x;
    const int seg = blockIdx.x;
    const int t = blockIdx.y;
    const int j_seg = seg * kRouterSegment;
    float w[kRouterSegment];
    const float* wp = w_router + (size_t)j_seg * E + min(lane, E - 1);   // lanes >= E read a valid column; never used
#pragma unroll
    for (int jj = 0; jj < kRouterSegment; ++jj) w[jj] = wp[(size_t)jj * E];
    float acc = 0.0f;
    if (IS_BF16) {
        const uint32_t* xp = (const uint32_t*)((const bf16_t*)x + (size_t)t * d + j_seg);
#pragma unroll
        for (int i = 0; i < kRouterSegment / 2; ++i) {
            const uint32_t p = xp[i];
            acc = __builtin_fmaf(__uint_as_float(p << 16), w[2 * i], acc);
            acc = __builtin_fmaf(__uint_as_float(p & 0xFFFF0000u), w[2 * i + 1], acc);
        }
    } else {
        const float* xp = (const float*)x + (size_t)t * d + j_seg;
#pragma unroll
        for (int i = 0; i < kRouterSegment; ++i) acc = __builtin_fmaf(xp[i], w[i], acc);
    }
    partial[((size_t)seg * T + t) * 64 + lane] = acc;
}

// The logits before the bias of tokens t[]: ordered sums of the segment partials; the loads of 8 segments are issued
// together (the adds stay in order).  A row of partials holds `pstride` floats; lanes past it hold no expert.
template <int TM>
__device__ __forceinline__ void sum_partials(const float* __restrict__ partial, int pstride, const int (&t)[TM], int T, int nseg,
                                             int lane, float (&total)[TM]) {
    const int col = min(lane, pstride - 1);
#pragma unroll
    for (int m = 0; m < TM; ++m) total[m] = partial[(size_t)t[m] * pstride + col];
    for (int sg0 = 1; sg0 < nseg; sg0 += 8) {
        float tmp[8][TM];
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int m = 0; m < TM; ++m)
                tmp[c][m] = partial[((size_t)min(sg0 + c, nseg - 1) * T + t[m]) * pstride + col];
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (sg0 + c < nseg) {
#pragma unroll
                for (int m = 0; m < TM; ++m) total[m] = total[m] + tmp[c][m];
            }
    }
}

// Selection for the TOK tokens of a workgroup of NW waves, one lane per expert (E <= 64); this wave's are m0 .. m0 + TM - 1
// with the logits (before the bias) `logit`: top-k and gates as pick_experts and gate_of give them.
//   Each selected (token, slot) also gets its rank among the workgroup's earlier assignments to the same expert (tokens
//   ascending), which is what makes the later scatter a stable counting sort without atomics.
template <int TOK, int TM, int NW>
__device__ __forceinline__ void select_experts(float (&logit)[TM], const float* __restrict__ bias, int m0, int tok0,
                                               int T, int E, int k, int32_t (*hit)[64], int32_t* __restrict__ topk_idx,
                                               float* __restrict__ gates, int32_t* __restrict__ local_rank,
                                               int32_t* __restrict__ blk_hist) {
    const int lane = threadIdx.x & 63;
    const bool owner = m0 < TOK;
    int32_t sel[TM];            // lane s (< k): expert in slot s
    float val[TM];              // lane s (< k): its logit
    bool taken[TM];             // lane e: the token selected expert e
    if (owner) {
        pick_experts<TM>(logit, bias, E, k, taken, sel, val);   // (rows past T hold the last row's logits; they are dropped below)
#pragma unroll
        for (int m = 0; m < TM; ++m) hit[m0 + m][lane] = (taken[m] && tok0 + m0 + m < T) ? 1 : 0;   // (hit is [TOK][64])
    }
    __syncthreads();
    if ((int)(threadIdx.x >> 6) == NW - 1) {
        int32_t h = 0;
#pragma unroll
        for (int m = 0; m < TOK; ++m) h += hit[m][lane];
        blk_hist[(size_t)blockIdx.x * 64 + lane] = h;
    }
    if (!owner) return;
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        const int t = tok0 + m0 + m;
        if (t >= T) break;
        const float g = gate_of(val[m], k);
        if (lane < k) {
            // rank among the block's earlier assignments to the same expert (tokens ascending), which is what makes the
            // later scatter a stable counting sort without atomics
            int32_t before = 0;
#pragma unroll
            for (int q = 0; q < TOK; ++q) before += q < m0 + m ? hit[q][sel[m]] : 0;
            const size_t a = (size_t)t * k + lane;
            topk_idx[a] = sel[m];
            gates[a] = g;
            local_rank[a] = before;
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// The segment chains of router_partial_mfma_kernel, router_topk_kernel and router_topk_lds_kernel run on the matrix cores: the fp32 MFMAs with a
// reduction length of ONE give every accumulator exactly one fused multiply-add per instruction (same bits as fmaf,
// denormals, infinities and NaN included), so the order above is kept at twice the rate of v_fma_f32.  Their blocks are
// used as a broadcast: one operand (CBSZ) is taken by all blocks from the lanes ABID names.
// ---------------------------------------------------------------------------------------------------------
constexpr int kNarrowRouterMaxE = 16;       // up to so many experts above kFineRouterMaxT tokens: partials of 16 columns, through memory
constexpr int kHalfRouterMaxT = 2048, kLdsRouterMaxT = 12288;
template <int N> struct IntC { static constexpr int value = N; };
template <typename F, int... N>
__device__ __forceinline__ void for_each_number(F& f, std::integer_sequence<int, N...>) { (f(IntC<N>{}), ...); }

// Eight consecutive elements of a row of x as loaded, and widened exactly.
template <bool IS_BF16> struct Octet;
template <> struct Octet<true> {
    u32x4_t p;
    __device__ __forceinline__ void load(const void* x, size_t i) { p = *(const u32x4_t*)((const bf16_t*)x + i); }
    __device__ __forceinline__ float get(int e) const {
        return __uint_as_float((e & 1) ? (p[e >> 1] & 0xFFFF0000u) : (p[e >> 1] << 16));
    }
};
template <> struct Octet<false> {
    f32x4_t p[2];
    __device__ __forceinline__ void load(const void* x, size_t i) {
        p[0] = *(const f32x4_t*)((const float*)x + i);
        p[1] = *(const f32x4_t*)((const float*)x + i + 4);
    }
    __device__ __forceinline__ float get(int e) const { return p[e >> 2][e & 3]; }
};

// router_topk_kernel (kSmallRouterMaxT < T <= kFineRouterMaxT): logits, top-k and gates of 4 tokens per workgroup of 16
// waves, one segment per wave and pass.  v_mfma_f32_4x4x1_16b_f32: the 16 blocks are 16 groups of 4 experts (lane =
// expert), W is read one 256-byte row per element of the reduction, and the 4 tokens are broadcast: a lane's 16 bytes of x
// are octet lane / 4 of token lane % 4.  The partials meet in LDS and are added in segment order by the wave that owns the
// token, which then selects its experts.  Bound by the 256 * d bytes of W that every workgroup pulls through its CU
// (31 B/clk: about 7 us at d = 2048), so it only pays while the workgroups are few.
// Measured against partials through memory and a top-k launch: 10.5 us against 11.1 + 14.3 us at T = 256, d = 2048, 64
// experts; 9.1 against 11.3 + 16.4 us at T = 777, d = 1280.  For T <= 64 the two launches are as fast (8.6 + 6.5 us at
// T = 64: more CUs share the reading of W), above 1024 workgroups of 4 tokens no longer fit the chip at once.
template <bool IS_BF16>
__device__ __forceinline__ void router_segment(const void* __restrict__ x, const float* __restrict__ w_router, int tok0, int T,
                                               int d, int E, int j0, int lane, float (*out)[64]) {
    typedef const __attribute__((address_space(1))) char* global_ptr;
    Octet<IS_BF16> xo;                           // rows past T re-read the last row; never used
    xo.load(x, (size_t)min(tok0 + (lane & 3), T - 1) * d + j0 + 8 * (lane >> 2));
    float w[2][32];                              // two chunks of 32 rows of W: one in use, one on its way
    const uint32_t off = (uint32_t)min(lane, E - 1) * 4u;                // lanes >= E read a valid column
    global_ptr row = (global_ptr)(w_router + (size_t)j0 * E);
    const size_t step = (size_t)E * 4;
    auto fetch_w = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            // the origin stays in scalar registers and is advanced: as 128 hoisted 64-bit products it spills
            asm volatile("" : "+s"(row));
            w[buf][i] = *(const __attribute__((address_space(1))) float*)(row + off);
            row += step;
        }
    };
    fetch_w(0);
    fetch_w(1);
    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
    float xf[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) xf[e] = xo.get(e);
    auto octet = [&](auto b) {                   // elements 8b .. 8b + 7 of the segment
        constexpr int B = decltype(b)::value;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(xf[e], w[(B / 4) & 1][8 * (B % 4) + e], acc, 4, B, 0);
    };
    auto chunk = [&](auto c) {
        constexpr int C = decltype(c)::value;
        octet(IntC<4 * C>{}); octet(IntC<4 * C + 1>{}); octet(IntC<4 * C + 2>{}); octet(IntC<4 * C + 3>{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (C < 2) fetch_w(C);         // the chunk after the next, into the registers just used
        __builtin_amdgcn_sched_barrier(0);
    };
    chunk(IntC<0>{}); chunk(IntC<1>{}); chunk(IntC<2>{}); chunk(IntC<3>{});
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i][lane] = acc[i];
}

template <bool IS_BF16>
__global__ void __launch_bounds__(1024)
router_topk_kernel(const void* __restrict__ x, const float* __restrict__ w_router, const float* __restrict__ bias, int T,
                   int d, int E, int k, int32_t* __restrict__ topk_idx, float* __restrict__ gates,
                   int32_t* __restrict__ local_rank, int32_t* __restrict__ blk_hist) {
    constexpr int NW = 16, TOK = 4;
    __shared__ float part[NW][TOK][64];
    __shared__ int32_t hit[TOK][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tok0 = blockIdx.x * TOK;
    const int nseg = d / kRouterSegment;
    float total[1] = {0.0f};
    for (int s0 = 0; s0 < nseg; s0 += NW) {
        const int seg = s0 + wave;
        if (seg < nseg) router_segment<IS_BF16>(x, w_router, tok0, T, d, E, seg * kRouterSegment, lane, part[wave]);
        __syncthreads();
        if (wave < TOK) {                        // the segments in order; the first partial is taken as is
            const int n = min(NW, nseg - s0);
            float p[NW];
#pragma unroll
            for (int s = 0; s < NW; ++s) p[s] = part[s][wave][lane];   // (rows past the last segment are not used)
            total[0] = s0 == 0 ? p[0] : total[0] + p[0];
#pragma unroll
            for (int s = 1; s < NW; ++s)
                if (s < n) total[0] = total[0] + p[s];
        }
        __syncthreads();
    }
    select_experts<TOK, 1, NW>(total, bias, wave, tok0, T, E, k, hit, topk_idx, gates, local_rank, blk_hist);
}

// router_topk_lds_kernel (kFineRouterMaxT < T <= kLdsRouterMaxT, more than kNarrowRouterMaxE experts): the same for TOK = 8 or 16 tokens
// per workgroup, so that W is pulled through a CU for enough of them.  A wave's segment of W comes to LDS in pieces of four rows, 16 bytes
// per lane straight from memory, kWRing of them on their way, and is read back one row per element of the reduction: lane = expert.
// The partials then take the ring's place.  Bound by the multiply-adds (6.9 us at T = 4096, d = 2048, 16 tokens on each CU) and the round
// trips before and after them; twice the pieces on their way change nothing, and two workgroups per CU (64 registers) spill: 24 instead of 20 us.
// Router and selection against partials through memory and a top-k launch, us, 64 experts, d 2048: T 1500, k 2 14.9 -> 10.9; T 2048, k 8
// 16.1 -> 12.1; T 4096, k 8 26.2 -> 19.9, k 1 22.7 -> 16.8; T 8192, k 2 34.5 -> 32.0; d 4096, T 4096 33.6 -> 28.1.  Up to
// kHalfRouterMaxT tokens 8 per workgroup put all CUs to work, above, W would be pulled twice through each.  A workgroup has its CU to itself, so what
// it gains is used up by the rounds: T 6000 31.1 / 31.2, T 12000 49.1 / 47.6, d 512 21.4 / 20.0, but T 20000, d 512 27.4 / 31.8, hence
// the line at kLdsRouterMaxT.
constexpr int kWRing = 4, kWPiece = 256;         // floats of a piece: four rows of at most 64
// The four rows of ring place SLOT at LDS byte addresses at[]: N younger pieces may still be on their way.  (Written out: the compiler
// would wait for all of them before a read that may touch the same array.)
template <int SLOT, int N>
__device__ __forceinline__ void read_piece(float (&w)[4], const uint32_t (&at)[4]) {
    asm volatile("s_waitcnt vmcnt(%9)\n\t"
                 "ds_read_b32 %0, %4 offset:%8\n\tds_read_b32 %1, %5 offset:%8\n\t"
                 "ds_read_b32 %2, %6 offset:%8\n\tds_read_b32 %3, %7 offset:%8\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "n"(SLOT * kWPiece * 4), "n"(N) : "memory");
}

template <bool IS_BF16, int TOK>
__global__ void __launch_bounds__(1024)
router_topk_lds_kernel(const void* __restrict__ x, const float* __restrict__ w_router, const float* __restrict__ bias, int T,
                       int d, int E, int k, int32_t* __restrict__ topk_idx, float* __restrict__ gates,
                       int32_t* __restrict__ local_rank, int32_t* __restrict__ blk_hist) {
    constexpr int NW = 16, G = TOK / 4, NP = kRouterSegment / 4;
    static_assert(TOK * 64 <= kWRing * kWPiece, "a wave's partials fit its part of the ring");
    __shared__ __attribute__((aligned(16))) float ring[NW][kWRing * kWPiece];
    __shared__ int32_t hit[TOK][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tok0 = blockIdx.x * TOK;
    const int nseg = d / kRouterSegment;
    float* own = ring[wave];
    uint32_t at[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)                  // lanes >= E read a valid column; never used
        at[r] = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float*)own + (uint32_t)(r * E + min(lane, E - 1)) * 4u;
    float total[1] = {0.0f};
    for (int s0 = 0; s0 < nseg; s0 += NW) {
        const int seg = s0 + wave, j0 = seg * kRouterSegment;
        if (seg < nseg) {
            Octet<IS_BF16> xo[G];                // rows past T re-read the last row; never used
#pragma unroll
            for (int g = 0; g < G; ++g) xo[g].load(x, (size_t)min(tok0 + 4 * g + (lane & 3), T - 1) * d + j0 + 8 * (lane >> 2));
            const float* wseg = w_router + (size_t)j0 * E;
            // (a piece is 16 * E bytes, one lane's 16 per expert; the lanes past them repeat the last)
            auto fetch = [&](int i) { load_to_lds(wseg, (uint32_t)min(lane, E - 1) * 16u, (uint32_t)i * (uint32_t)E * 16u, own + (i % kWRing) * kWPiece); };
#pragma unroll
            for (int i = 0; i < kWRing; ++i) fetch(i);
            float xf[G][8];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < 8; ++e) xf[g][e] = xo[g].get(e);
            f32x4_t acc[G];
#pragma unroll
            for (int g = 0; g < G; ++g) acc[g] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            auto piece = [&](auto i_tag) {       // elements 4i .. 4i + 3 of the segment
                constexpr int I = decltype(i_tag)::value;
                float w[4];
                read_piece<I % kWRing, (NP - 1 - I < kWRing - 1 ? NP - 1 - I : kWRing - 1)>(w, at);
                if constexpr (I + kWRing < NP) fetch(I + kWRing);
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        acc[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(xf[g][(4 * I + r) % 8], w[r], acc[g], 4, I / 2, 0);
            };
            for_each_number(piece, std::make_integer_sequence<int, NP>{});
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) own[(4 * g + i) * 64 + lane] = acc[g][i];
        }
        __syncthreads();
        if (wave < TOK) {                        // the segments in order; the first partial is taken as is
            const int n = min(NW, nseg - s0);
            float p[NW];
#pragma unroll
            for (int s = 0; s < NW; ++s) p[s] = ring[s][wave * 64 + lane];   // (rows past the last segment are not used)
            total[0] = s0 == 0 ? p[0] : total[0] + p[0];
#pragma unroll
            for (int s = 1; s < NW; ++s)
                if (s < n) total[0] = total[0] + p[s];
        }
        __syncthreads();
    }
    select_experts<TOK, 1, NW>(total, bias, wave, tok0, T, E, k, hit, topk_idx, gates, local_rank, blk_hist);
}

// router_partial_mfma_kernel (T > kFineRouterMaxT; with more than kNarrowRouterMaxE experts T > kLdsRouterMaxT): segment partials of 8
// waves' tokens; a workgroup takes one segment, whose W (512 * E bytes) it keeps in LDS for all its tokens.
//   NARROW = false: v_mfma_f32_16x16x1_4b_f32 as four groups of 16 experts x 16 tokens; the tokens (rows) are broadcast: a
//                   lane holds octets 4o + lane / 16 of token lane % 16.  16 tokens per wave; partial rows of 64 floats.
//   NARROW = true (E <= 16): four groups of 16 tokens x 16 experts; the experts (rows) are broadcast: a lane holds
//                   W[4j + lane / 16][lane % 16], and all of its own token's segment.  64 tokens per wave, rows of 16.
// Bound by the multiply-adds (2*T*d*64 flop at 157 TFLOP/s: 6.9 us at T = 4096, d = 2048; with E <= 16 by reading x).
// Measured against register-tiled v_fma_f32 kernels: 19.0 us against 27.4 at T = 4096, d = 2048, 64 experts (32.7 against
// 41.9 at T = 8192, 9.9 against 21.7 at T = 2048); NARROW 16.5 us against 20.4 at T = 4096, d = 4096, 8 experts.  W is
// read from LDS eight registers ahead (one read per multiply-add, waited for at once, took 22.7 us).
template <bool IS_BF16, bool NARROW>
__global__ void __launch_bounds__(512)
router_partial_mfma_kernel(const void* __restrict__ x, const float* __restrict__ w_router, int T, int d, int E,
                           float* __restrict__ partial) {
    constexpr int TW = NARROW ? 64 : 16;         // tokens per wave
    typedef __attribute__((ext_vector_type(16))) float f32x16;
    __shared__ __attribute__((aligned(16))) float ws[kRouterSegment * (NARROW ? 16 : 64)];   // [128][16 or 64]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int seg = blockIdx.y, j0 = seg * kRouterSegment;
    const int t0 = (blockIdx.x * 8 + wave) * TW;
    const int l16 = lane & 15, q = lane >> 4;

    constexpr int NO = NARROW ? 16 : 4;
    Octet<IS_BF16> xo[NO];                       // rows past T re-read the last row; never stored
    const size_t xrow = (size_t)min(t0 + (NARROW ? lane : l16), T - 1) * d + j0;
#pragma unroll
    for (int o = 0; o < NO; ++o) xo[o].load(x, xrow + 8 * (NARROW ? o : 4 * o + q));
    constexpr int EW = NARROW ? 16 : 64, NL = kRouterSegment * EW / 512;
    float wst[NL];
#pragma unroll
    for (int p = 0; p < NL; ++p) {               // columns past E repeat the last one; never used
        const int i = tid + 512 * p;
        wst[p] = w_router[(size_t)(j0 + i / EW) * E + min(i % EW, E - 1)];
    }
#pragma unroll
    for (int p = 0; p < NL; ++p) ws[tid + 512 * p] = wst[p];
    __syncthreads();

    // W in groups of NG registers, the next group read from LDS while the current one is multiplied.  A register holds
    // element k of column `lane`, or (NARROW) elements 4j + 0..3 of the 16 columns.
    constexpr int NR = kRouterSegment * EW / 64, NG = 8;
    // (column l16 of block q is expert 4 * l16 + q: the four blocks of an accumulator then hold four consecutive experts)
    const int wcol = NARROW ? lane : 4 * l16 + q;
    f32x16 acc = {};
    float w[2][NG];
    auto read_w = [&](int g) {
#pragma unroll
        for (int i = 0; i < NG; ++i) w[g & 1][i] = ws[(g * NG + i) * 64 + wcol];
    };
    read_w(0);
#pragma unroll
    for (int g = 0; g < NR / NG; ++g) {
        if (g + 1 < NR / NG) read_w(g + 1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NARROW) {
#pragma unroll
            for (int i = 0; i < NG; ++i) {       // elements 4j .. 4j + 3 of the segment, j = NG * g + i
                const Octet<IS_BF16>& o = xo[(NG * g + i) >> 1];
                acc = __builtin_amdgcn_mfma_f32_16x16x1f32(w[g & 1][i], o.get(4 * (i & 1)), acc, 2, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x1f32(w[g & 1][i], o.get(4 * (i & 1) + 1), acc, 2, 1, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x1f32(w[g & 1][i], o.get(4 * (i & 1) + 2), acc, 2, 2, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x1f32(w[g & 1][i], o.get(4 * (i & 1) + 3), acc, 2, 3, 0);
            }
        } else {
            const Octet<IS_BF16>& o = xo[g >> 2];   // octet g: lanes 16 * (g % 4) .. of register g / 4
#pragma unroll
            for (int e = 0; e < NG; ++e) {
                if ((g & 3) == 0) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(o.get(e), w[g & 1][e], acc, 2, 0, 0);
                if ((g & 3) == 1) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(o.get(e), w[g & 1][e], acc, 2, 1, 0);
                if ((g & 3) == 2) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(o.get(e), w[g & 1][e], acc, 2, 2, 0);
                if ((g & 3) == 3) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(o.get(e), w[g & 1][e], acc, 2, 3, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // accumulator element 4b + i of a lane: row 4 * (lane / 16) + i, column lane % 16 of block b
    float* out = partial + ((size_t)seg * T) * (NARROW ? 16 : 64);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if constexpr (NARROW) {                  // rows are experts, columns tokens
            const int t = t0 + 16 * b + l16;
            if (t < T) *(f32x4_t*)(out + (size_t)t * 16 + 4 * q) = f32x4_t{acc[4 * b], acc[4 * b + 1], acc[4 * b + 2], acc[4 * b + 3]};
        } else {                                 // rows are tokens: token 4q + b of the wave's, experts 4 * l16 + 0..3
            const int t = t0 + 4 * q + b;
            if (t < T) *(f32x4_t*)(out + (size_t)t * 64 + 4 * l16) = f32x4_t{acc[b], acc[4 + b], acc[8 + b], acc[12 + b]};
        }
    }
}

// topk_kernel: ordered sum of the segment partials (rows of `pstride` floats) and the selection, TOK tokens per workgroup
// of NW waves.
template <int TOK, int NW>
__global__ void __launch_bounds__(NW * 64)
topk_kernel(const float* __restrict__ partial, int pstride, const float* __restrict__ bias, int T, int nseg, int E, int k,
            int32_t* __restrict__ topk_idx, float* __restrict__ gates, int32_t* __restrict__ local_rank,
            int32_t* __restrict__ blk_hist) {
    constexpr int TM = TOK / NW;
    __shared__ int32_t hit[TOK][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tok0 = blockIdx.x * TOK;
    int t[TM];
    float total[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) t[m] = min(tok0 + wave * TM + m, T - 1);
    sum_partials<TM>(partial, pstride, t, T, nseg, lane, total);
    select_experts<TOK, TM, NW>(total, bias, wave * TM, tok0, T, E, k, hit, topk_idx, gates, local_rank, blk_hist);
}

// ---------------------------------------------------------------------------------------------------------
// permute_kernel (T > kFusedTailMaxT): the stable counting sort from the block histograms of the selection.  A workgroup of
// 16 waves scatters the assignments of its router blocks, kPermuteBlocks at a time: position of an assignment = offset of its
// expert + assignments to it in earlier blocks + its rank in the block.  Every workgroup sums all histograms itself (256 bytes
// per block, from the cache): one launch where a one-workgroup scan had to come first.  The first one also writes the counts,
// the offsets and the tiles of the grouped GEMMs.  Bound by latency: 5.6 us at 4096 tokens and 6.6 at 8192 against 5.9 + 5.7
// and 10.2 + 5.8 us for scan and scatter, 6.5 us against 8.8 (scan and scatter in one workgroup) at 777.
// What all workgroups read together grows with the square of the blocks.  Above kPermuteDirectBlocks of them hist_sum_kernel
// first adds each workgroup's blocks up, and `sums` holds one row per workgroup instead of one per block: a launch more, and
// linear.  The whole routing stage with either (d 128, 8 experts, k = 1, us): 8192 tokens 22 / 22, 16384 27 / 24, 65536 67 / 40,
// 131072 177 / 51 (scan and scatter 169), 1048576 8545 / 287 (1225).
// ---------------------------------------------------------------------------------------------------------
constexpr int kPermuteBlocks = 8;

__global__ void __launch_bounds__(1024)
hist_sum_kernel(const int32_t* __restrict__ blk_hist, int nblk, int blocks, int32_t* __restrict__ sums) {
    __shared__ int32_t s_part[16][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b0 = blockIdx.x * blocks, b1 = min(b0 + blocks, nblk);
    int32_t total = 0;
    for (int b = b0 + wave; b < b1; b += 16) total += blk_hist[(size_t)b * 64 + lane];
    s_part[wave][lane] = total;
    __syncthreads();
    if (wave != 0) return;
    total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) total += s_part[w][lane];
    sums[(size_t)blockIdx.x * 64 + lane] = total;
}

// `sums`: nsums rows of 64, one per router block (a workgroup owns kPermuteBlocks of them) or one per workgroup.
__global__ void __launch_bounds__(1024)
permute_kernel(const int32_t* __restrict__ blk_hist, int nblk, const int32_t* __restrict__ sums, int nsums, int blocks, int E,
               WorkPlan plan, int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* __restrict__ sched,
               const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ local_rank, int T, int k, int tokens_per_block,
               int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm, int32_t* __restrict__ row_token) {
    __shared__ int32_t s_total[16][64], s_before[16][64];
    __shared__ int32_t s_base[kPermuteBlocks][64];      // first position of expert e's assignments in block b + i
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b0 = blockIdx.x * blocks, b1 = min(b0 + blocks, nblk);
    const int first = nsums == nblk ? b0 : blockIdx.x;  // the first row of `sums` that is this workgroup's
    int32_t total = 0, before = 0;                      // of the rows this wave sums; of those among them before `first`
    for (int b = wave; b < nsums; b += 16 * 8) {
        int32_t h[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) h[u] = sums[(size_t)min(b + 16 * u, nsums - 1) * 64 + lane];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int32_t v = b + 16 * u < nsums ? h[u] : 0;
            total += v;
            before += b + 16 * u < first ? v : 0;
        }
    }
    s_total[wave][lane] = total;
    s_before[wave][lane] = before;
    __syncthreads();
    int32_t pos = 0;                                    // wave 0: the next position of expert `lane`
    if (wave == 0) {
        total = before = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            total += s_total[w][lane];
            before += s_before[w][lane];
        }
        pos = wave_inclusive_sum(total) - total + before;
    } else if (wave == 1 && blockIdx.x == 0) {
        total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) total += s_total[w][lane];
        write_work_list(total, E, plan, counts, offsets, sched);
    }
    for (int b = b0; b < b1; b += kPermuteBlocks) {
        if (wave == 0) {
            int32_t own[kPermuteBlocks];
#pragma unroll
            for (int i = 0; i < kPermuteBlocks; ++i) own[i] = blk_hist[(size_t)min(b + i, nblk - 1) * 64 + lane];
#pragma unroll
            for (int i = 0; i < kPermuteBlocks; ++i) {
                s_base[i][lane] = pos;
                pos += own[i];
            }
        }
        __syncthreads();
        const int a0 = b * tokens_per_block * k, a1 = min(min(b + kPermuteBlocks, b1) * tokens_per_block, T) * k;
        for (int a = a0 + threadIdx.x; a < a1; a += 1024) {
            const int e = topk_idx[a];
            const int t = a / k;
            const int at = s_base[t / tokens_per_block - b][e] + local_rank[a];
            perm[at] = a;
            inv_perm[a] = at;
            row_token[at] = t;
        }
        __syncthreads();                                // s_base has been read
    }
}

// ---------------------------------------------------------------------------------------------------------
// topk_scan_kernel (decode-sized batches, T <= kFusedTailMaxT): ONE workgroup of 16 waves does everything after the
// segment partials -- the top-k and gates of every token (one token per wave per pass, tokens ascending), the
// per-expert counts, offsets and tile schedule, and the scatter.  With all tokens in one workgroup the stable
// counting sort needs no block histograms in memory: an assignment's position is offsets[e] + (assignments to e by
// earlier tokens), kept in LDS.  Saves two dependent launches on the latency-bound path.  (`sched` may lie in the memory of
// `partial`: it is written after the last barrier behind the reads.)
// ---------------------------------------------------------------------------------------------------------
constexpr int kFusedTailMaxA = kFusedTailMaxT * 64;   // assignments (k <= E <= 64)

__global__ void __launch_bounds__(1024)
topk_scan_kernel(const float* partial, const float* __restrict__ bias, int T, int nseg, int E, int k,
                 WorkPlan plan, int32_t* __restrict__ topk_idx, float* __restrict__ gates,
                 int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* sched,
                 int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                 int32_t* __restrict__ row_token) {
    __shared__ int32_t wave_hit[16][64];        // this pass: 1 if the wave's token selected expert e
    __shared__ int32_t s_seen[64];              // assignments to expert e by the tokens of earlier passes
    __shared__ int32_t s_off[64];
    __shared__ uint8_t s_e[kFusedTailMaxA];     // expert of assignment a
    __shared__ int16_t s_rank[kFusedTailMaxA];  // assignments to that expert by earlier tokens
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave == 0) s_seen[lane] = 0;
    __syncthreads();
    for (int t0 = 0; t0 < T; t0 += 16) {
        const int t = t0 + wave;
        const bool live = t < T;                // wave-uniform
        int32_t sel[1] = {0};
        bool hit[1] = {false};
        if (live) {
            const int tt[1] = {t};
            float sum[1], val[1];
            sum_partials<1>(partial, 64, tt, T, nseg, lane, sum);
            pick_experts<1>(sum, bias, E, k, hit, sel, val);
            const float g = gate_of(val[0], k);
            if (lane < k) {
                const size_t a = (size_t)t * k + lane;
                topk_idx[a] = sel[0];
                gates[a] = g;
                s_e[a] = (uint8_t)sel[0];
            }
        }
        wave_hit[wave][lane] = hit[0] ? 1 : 0;
        __syncthreads();
        if (live && lane < k) {
            int32_t before = s_seen[sel[0]];
            for (int w = 0; w < wave; ++w) before += wave_hit[w][sel[0]];
            s_rank[t * k + lane] = (int16_t)before;
        }
        __syncthreads();
        if (wave == 0) {
            int32_t h = 0;
#pragma unroll
            for (int w = 0; w < 16; ++w) h += wave_hit[w][lane];
            s_seen[lane] += h;
        }
        __syncthreads();
    }
    if (wave == 0) s_off[lane] = write_work_list(s_seen[lane], E, plan, counts, offsets, sched);
    __syncthreads();
    const int A = T * k;
    for (int a = threadIdx.x; a < A; a += 1024) {
        const int pos = s_off[s_e[a]] + s_rank[a];
        perm[pos] = a;
        inv_perm[a] = pos;
        row_token[pos] = a / k;
    }
}

// ---------------------------------------------------------------------------------------------------------
// route_small_kernel (T <= kSmallRouterMaxT, at most kSmallRouteSegs segments): the whole routing in ONE workgroup of 16 waves, four
// tokens each.  A segment's W (at most 32 KB) goes through LDS once for all of them; v_mfma_f32_4x4x1_16b_f32 as in
// router_topk_kernel leaves a token's partial with lane = expert, where it is added up and selected from.  The counting sort
// needs no histograms: an expert's tokens are 64 bits.
// Routing stage with events, one launch against three: 64 tokens, d 128, k = 2 11.1 us against 12.5.  One CU does all the work, at 1 us
// per k and 2.7 us per further segment for 64 tokens: k = 6 15.1 / 13.2, d 256, k = 4 15.8 / 13.3; hence the line at 192.  A fourth
// segment costs more than it saves (8 fp32 layers, d 512, 1 to 12 tokens 157 to 188 us against 143 to 173), the third pays above 16
// tokens (d 384, 17 tokens, 8 experts 160 / 163, 64 experts 166 / 182).  Up to 16 tokens one launch replaces two only: called from the host
// it is the faster one (d 256, 2 tokens, k 8 148 / 160; d 384, 2 tokens, k 1 144 / 155), in a replayed graph the selection's k rounds
// and the third segment cost 3 to 5 % (148 / 140, 144 / 140); few tokens of such narrow layers come from the host.
// Up to 16 experts a row of 16 lanes is enough for a token, so a wave selects from its four at once, a quarter of the work per k: 64 tokens, d 128,
// k 2 9.0 -> 6.7 us, 32 tokens, k 4 7.0 -> 4.9.  The line moves with it, one launch against three: d 128, 64 tokens, k 4 7.0 / 9.9, 16 experts,
// k 8 8.5 / 10.6; d 256, 64 tokens, k 4 10.0 / 11.0, k 8 10.4 / 10.8; d 384, 32 tokens, k 4 8.1 / 9.5, k 8 9.8 / 10.4, but 64 tokens, k 2 12.5 / 10.2.
// Up to 16 tokens it pays in a replayed graph too (4 bf16 layers of d 384, two launches against one, replayed, from the host): 16 tokens, 8
// experts, k 8 81.1 / 77.5, 86.2 / 76.7; 16 experts, k 16 96.5 / 91.6, 95.2 / 90.6; 9 tokens, k 16 91.3 / 88.7, 90.0 / 86.8.
// ---------------------------------------------------------------------------------------------------------
constexpr int kSmallRouteSegs = 3;
static bool route_small(int T, int k, int nseg, int E) {
    if (T > kSmallRouterMaxT || nseg > kSmallRouteSegs) return false;
    return E <= kNarrowRouterMaxE ? T * (k + 12 * (nseg - 1)) <= 1024 : T * (k + 3 * (nseg - 1)) <= 192;
}

template <bool IS_BF16>
__global__ void __launch_bounds__(1024)
route_small_kernel(const void* __restrict__ x, const float* __restrict__ w_router, const float* __restrict__ bias, int T, int d,
                   int E, int k, WorkPlan plan, int32_t* __restrict__ topk_idx, float* __restrict__ gates,
                   int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* __restrict__ sched,
                   int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm, int32_t* __restrict__ row_token) {
    __shared__ __attribute__((aligned(16))) float ws[kRouterSegment * 64];
    __shared__ uint8_t s_bits[16][64];           // which of a wave's four tokens selected expert e
    __shared__ uint64_t s_tokens[64];            // the tokens of expert e
    __shared__ int32_t s_off[64];
    __shared__ uint8_t s_sel[kSmallRouterMaxT * 64];   // the expert of assignment a
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tok0 = wave * 4;
    const int nseg = d / kRouterSegment;
    float wst[8];
    Octet<IS_BF16> xo;                                                  // rows past T re-read the last row; never used
    auto fetch = [&](int seg) {
        const float* wp = w_router + (size_t)(seg * kRouterSegment + wave) * E + min(lane, E - 1);   // lanes >= E read a valid column
#pragma unroll
        for (int p = 0; p < 8; ++p) wst[p] = wp[(size_t)16 * p * E];
        xo.load(x, (size_t)min(tok0 + (lane & 3), T - 1) * d + seg * kRouterSegment + 8 * (lane >> 2));
    };
    fetch(0);
    float total[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int seg = 0; seg < nseg; ++seg) {
#pragma unroll
        for (int p = 0; p < 8; ++p) ws[tid + 1024 * p] = wst[p];
        float xf[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) xf[e] = xo.get(e);
        __syncthreads();
        if (seg + 1 < nseg) fetch(seg + 1);
        if (tok0 < T) {
            f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
            auto octet = [&](auto b) {           // elements 8B .. 8B + 7 of the segment
                constexpr int B = decltype(b)::value;
                float w[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = ws[(8 * B + e) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(xf[e], w[e], acc, 4, B, 0);
            };
            octet(IntC<0>{}); octet(IntC<1>{}); octet(IntC<2>{}); octet(IntC<3>{});
            octet(IntC<4>{}); octet(IntC<5>{}); octet(IntC<6>{}); octet(IntC<7>{});
            octet(IntC<8>{}); octet(IntC<9>{}); octet(IntC<10>{}); octet(IntC<11>{});
            octet(IntC<12>{}); octet(IntC<13>{}); octet(IntC<14>{}); octet(IntC<15>{});
#pragma unroll
            for (int m = 0; m < 4; ++m) total[m] = seg == 0 ? acc[m] : total[m] + acc[m];   // the first partial is taken as is
        }
        __syncthreads();                         // ws has been read
    }
    uint32_t bits = 0;
    if (tok0 < T && E <= kNarrowRouterMaxE) {    // a row of 16 lanes has a token's experts: the four tokens at once, the same values and order
        const int l16 = lane & 15, t = tok0 + (lane >> 4);
        float v = __shfl(total[0], l16);
#pragma unroll
        for (int m = 1; m < 4; ++m) {
            const float o = __shfl(total[m], l16);
            v = lane >> 4 == m ? o : v;
        }
        if (bias != nullptr) v = v + bias[min(l16, E - 1)];
        v = v == v ? v : -INFINITY;              // (as in pick_experts)
        bool open = l16 < E;
        int32_t sel = 0;
        float val = -INFINITY;
        for (int s = 0; s < k; ++s) {
            const float mx = row_max(open ? v : -INFINITY);
            const uint32_t holds = (uint32_t)(__ballot(open && v == mx) >> (lane & 48)) & 0xFFFFu;
            const int e_star = __builtin_ctz(holds);
            if (l16 == e_star) open = false;
            if (l16 == s) { sel = e_star; val = mx; }
        }
        const float ex = l16 < k ? __expf(val - __shfl(val, lane & 48)) : 0.0f;
        const float g = ex / row_sum(ex);
        if (t < T && l16 < k) {
            topk_idx[t * k + l16] = sel;
            gates[t * k + l16] = g;
            s_sel[t * k + l16] = (uint8_t)sel;
        }
        const uint64_t taken = __ballot(t < T && l16 < E && !open) >> l16;
        if (lane < 16) bits = (uint32_t)(taken & 1) | (uint32_t)(taken >> 15 & 2) | (uint32_t)(taken >> 30 & 4) | (uint32_t)(taken >> 45 & 8);
    } else if (tok0 < T) {
        bool taken[4];
        int32_t sel[4];
        float val[4];
        pick_experts<4>(total, bias, E, k, taken, sel, val);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int t = tok0 + m;
            if (t >= T) break;
            bits |= taken[m] ? 1u << m : 0u;
            const float g = gate_of(val[m], k);
            if (lane < k) {
                topk_idx[t * k + lane] = sel[m];
                gates[t * k + lane] = g;
                s_sel[t * k + lane] = (uint8_t)sel[m];
            }
        }
    }
    s_bits[wave][lane] = (uint8_t)bits;
    __syncthreads();
    if (wave == 0) {
        uint64_t tokens = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) tokens |= (uint64_t)s_bits[w][lane] << (4 * w);
        s_tokens[lane] = tokens;
        s_off[lane] = write_work_list(__popcll(tokens), E, plan, counts, offsets, sched);
    }
    __syncthreads();
    for (int a = tid; a < T * k; a += 1024) {
        const int t = a / k, e = s_sel[a];
        const int at = s_off[e] + __popcll(s_tokens[e] & ((1ull << t) - 1));
        perm[at] = a;
        inv_perm[a] = at;
        row_token[at] = t;
    }
}

// ---------------------------------------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------------------------------------

static bool lds_router(int T, int E) { return T > kFineRouterMaxT && T <= kLdsRouterMaxT && E > kNarrowRouterMaxE; }
static int router_tokens_per_block(int T, int E) {
    if (T <= kSmallRouterMaxT) return 8;
    if (T <= kFineRouterMaxT) return 4;
    return lds_router(T, E) && T <= kHalfRouterMaxT ? 8 : 16;
}

template <bool IS_BF16>
static hipError_t launch_partials(const RoutingArgs& a, hipStream_t s) {
    const int nseg = a.d / kRouterSegment;
    if (a.T <= kSmallRouterMaxT)
        hipLaunchKernelGGL(router_partial_small_kernel<IS_BF16>, dim3(nseg, a.T), dim3(64), 0, s, a.x, a.w_router, a.T, a.d,
                           a.E, a.partial);
    else if (a.E <= kNarrowRouterMaxE)
        hipLaunchKernelGGL((router_partial_mfma_kernel<IS_BF16, true>), dim3((a.T + 511) / 512, nseg), dim3(512), 0, s, a.x,
                           a.w_router, a.T, a.d, a.E, a.partial);
    else
        hipLaunchKernelGGL((router_partial_mfma_kernel<IS_BF16, false>), dim3((a.T + 127) / 128, nseg), dim3(512), 0, s, a.x,
                           a.w_router, a.T, a.d, a.E, a.partial);
    return hipGetLastError();
}

hipError_t launch_router_partials(const RoutingArgs& a, hipStream_t s) {
    return a.is_bf16 ? launch_partials<true>(a, s) : launch_partials<false>(a, s);
}

hipError_t launch_routing(const RoutingArgs& a, hipStream_t s) {
    const int nseg = a.d / kRouterSegment;
    const int tb = router_tokens_per_block(a.T, a.E);
    const int nblk = (a.T + tb - 1) / tb;
    hipError_t err;
    if (route_small(a.T, a.k, nseg, a.E)) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(1), dim3(1024), 0, s, a.x, a.w_router, a.bias, a.T, a.d, a.E, a.k, a.plan, a.topk_idx, a.gates,
                               a.counts, a.offsets, a.sched, a.perm, a.inv_perm, a.row_token);
        };
        if (a.is_bf16) launch(route_small_kernel<true>);
        else launch(route_small_kernel<false>);
        return hipGetLastError();
    }
    if (a.T > kSmallRouterMaxT && a.T <= kFineRouterMaxT) {
        if (a.is_bf16)
            hipLaunchKernelGGL(router_topk_kernel<true>, dim3(nblk), dim3(1024), 0, s, a.x, a.w_router, a.bias, a.T, a.d, a.E,
                               a.k, a.topk_idx, a.gates, a.local_rank, a.blk_hist);
        else
            hipLaunchKernelGGL(router_topk_kernel<false>, dim3(nblk), dim3(1024), 0, s, a.x, a.w_router, a.bias, a.T, a.d, a.E,
                               a.k, a.topk_idx, a.gates, a.local_rank, a.blk_hist);
        err = hipGetLastError();
    } else if (lds_router(a.T, a.E)) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(nblk), dim3(1024), 0, s, a.x, a.w_router, a.bias, a.T, a.d, a.E, a.k, a.topk_idx, a.gates,
                               a.local_rank, a.blk_hist);
        };
        if (tb == 8) {
            if (a.is_bf16) launch(router_topk_lds_kernel<true, 8>);
            else launch(router_topk_lds_kernel<false, 8>);
        } else {
            if (a.is_bf16) launch(router_topk_lds_kernel<true, 16>);
            else launch(router_topk_lds_kernel<false, 16>);
        }
        err = hipGetLastError();
    } else {
        err = launch_router_partials(a, s);
        if (err != hipSuccess) return err;
        if (a.T <= kFusedTailMaxT) {
            hipLaunchKernelGGL(topk_scan_kernel, dim3(1), dim3(1024), 0, s, a.partial, a.bias, a.T, nseg, a.E, a.k,
                               a.plan, a.topk_idx, a.gates, a.counts, a.offsets, a.sched, a.perm, a.inv_perm, a.row_token);
            return hipGetLastError();
        }
        if (tb == 8)
            hipLaunchKernelGGL((topk_kernel<8, 8>), dim3(nblk), dim3(512), 0, s, a.partial, 64, a.bias, a.T, nseg, a.E, a.k,
                               a.topk_idx, a.gates, a.local_rank, a.blk_hist);
        else
            hipLaunchKernelGGL((topk_kernel<16, 8>), dim3(nblk), dim3(512), 0, s, a.partial, a.E <= kNarrowRouterMaxE ? 16 : 64,
                               a.bias, a.T, nseg, a.E, a.k, a.topk_idx, a.gates, a.local_rank, a.blk_hist);
        err = hipGetLastError();
    }
    if (err != hipSuccess) return err;
    const int32_t* sums = a.blk_hist;
    int nsums = nblk, blocks = kPermuteBlocks;
    if (nblk > kPermuteDirectBlocks) {
        blocks = (nblk + kHistSums * kPermuteBlocks - 1) / (kHistSums * kPermuteBlocks) * kPermuteBlocks;
        nsums = (nblk + blocks - 1) / blocks;
        sums = a.hist_sums;
        hipLaunchKernelGGL(hist_sum_kernel, dim3(nsums), dim3(1024), 0, s, a.blk_hist, nblk, blocks, a.hist_sums);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL(permute_kernel, dim3((nblk + blocks - 1) / blocks), dim3(1024), 0, s, a.blk_hist, nblk, sums, nsums, blocks,
                       a.E, a.plan, a.counts, a.offsets, a.sched, a.topk_idx, a.local_rank, a.T, a.k, tb, a.perm, a.inv_perm,
                       a.row_token);
    return hipGetLastError();
}

}  // namespace lexi
