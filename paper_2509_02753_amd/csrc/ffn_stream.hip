// Expert FFN, weight-streaming schedule for decode-sized batches (a few rows per expert): the time goes into reading
// each touched expert's weights from HBM once, so the kernel is built around memory-level parallelism, not MFMA rate.
//
// A workgroup owns ONE unit of 16 output features of one token tile (gate/up: 16 gate rows + the 16 matching up
// rows) and splits the reduction dimension over its 4 or 8 waves.  A wave streams its part of the unit's packed
// 16 x 32 weight blocks -- 1 KB fully coalesced loads, many in flight -- and multiplies each against the tile's
// token blocks (16 tokens x 32 K, read straight from the token rows, which stay cache-resident) with
// v_mfma_f32_16x16x32_bf16.  The partial accumulators are added in wave order through LDS (fixed order: same
// bits every run), then the epilogue of the tile schedule's kernel applies: silu(gate)*up -> bf16, or fp32 rows.
// (stream_unit in ffn_common.hpp: the tile kernel's launches take such units too.)
#include "ffn_common.hpp"
#include "routing_common.hpp"

namespace lexi {

// Registers of the loads on their way (stream_blocks).  The more the fewer waves fit: with four per SIMD (128 registers) 64 for the down
// GEMM, 48 beside the selection.  Down, us, 96 and three waves / 64 and four: 16 tokens, k 6 31.2 / 30.2, 64 experts without bias 53.0 / 51.3, 32 tokens,
// K 14336 163 / 157; select_gateup_kernel, 96 and three waves / 60 / 48: 16 tokens, k 2 28.7 / 29.6 / 28.3, k 6 57.8 / 58.3 / 56.9, 10
// tokens of d 1024 19.6 / 17.1 / 17.0.
constexpr int kStreamRegs = 64, kSelectStreamRegs = 48;

// TWO: a second job; else a grid of units x tiles (most workgroups of a launch that uses few experts end at once, and neither choose
// a job nor divide before they do).
template <bool GATEUP, int NW, bool TWO>
__global__ void __launch_bounds__(NW * 64, GATEUP ? 2 : 4)
ffn_stream_kernel(FfnJob routed, FfnJob shared) {
    // (a streaming shared expert has at most 64 rows, and so has every expert beside it)
    constexpr int MAXB = TWO ? 4 : 8;
    __shared__ __attribute__((aligned(16))) f32x4_t red[TWO && NW == 4 ? stream_eight_lds<GATEUP>(MAXB) : NW * 2 * 64];
    int unit = blockIdx.x, tile = blockIdx.y;
    const FfnJob j = TWO ? pick_job(routed, shared, unit) : routed;
    if (TWO) {
        const int units = j.features >> 4, block = unit;
        tile = block / units;
        unit = block - tile * units;
    }
    TileInfo ti;
    if (!fetch_tile<GATEUP ? 0 : 1>(j, tile, ti)) return;
    auto row_of = [&](int r) { return j.row_token ? j.row_token[ti.row0 + r] : ti.row0 + r; };
    if (TWO) stream_unit_of<GATEUP, NW, MAXB, kStreamRegs>(j, ti, unit, red, row_of);
    else stream_unit<GATEUP, NW, MAXB, kStreamRegs>(j, ti, unit, (f32x4_t(*)[2][64])red, row_of);
}

// ---------------------------------------------------------------------------------------------------------
// select_gateup_kernel (at most kSelectMaxT tokens): the routing behind the router's partials costs a launch (4.7 us in a replayed
// graph) for a microsecond of work.  Here every workgroup of the gate/up launch selects the tokens' experts for itself, from
// partials that every one of them reads (4 KB a token at d = 2048), which takes the place of reading the work list: the experts of
// a token are 64 bits, so counts, offsets, an expert's tokens and the tile's expert are a few bit operations.  One workgroup
// writes the routing for the launches behind.  The workgroups take units of 16 features in steps of the grid, at most
// kSelectBlocks of them (most tokens use far fewer experts than they might), the shared expert's come first.
// Whole calls of 8 layers when it was made (us): one token, k 2 to 6 302 -> 265; 8 tokens, k = 6 643 -> 590; 16 tokens, k = 2 466 -> 424,
// k = 6 829 -> 798, k = 8 without a shared expert 1231 -> 1203.  What every workgroup reads grows with T * d, but so does what it streams:
// 10 to 16 tokens, k 4 to 8, d 3072 1 to 3 % less than with the launch, d 4096 to 8192 -1 to +2 %.
// ---------------------------------------------------------------------------------------------------------
constexpr int kSelectBlocks = 1024;

struct SelectArgs {
    const float *partial, *bias;
    int T, nseg, E, k;
    int32_t *topk_idx, *counts, *offsets, *perm, *inv_perm, *row_token;
    float* gates;
};

template <int NW, int MAXT>
__global__ void __launch_bounds__(NW * 64, 4)
select_gateup_kernel(FfnJob routed, FfnJob shared, SelectArgs r) {
    __shared__ __attribute__((aligned(16))) f32x4_t red[8 * 2 * 64];   // (of stream_unit_eight, or of eight waves)
    __shared__ uint64_t s_mask[MAXT];
    __shared__ uint8_t s_sel[MAXT][64];
    __shared__ int32_t s_off[64];
    const int lane = threadIdx.x & 63;
    if ((int)blockIdx.x < shared.blocks) {
        const int units = shared.features >> 4;
        if ((int)blockIdx.x < units) stream_unit_of<true, NW, 1, kSelectStreamRegs>(shared, TileInfo{0, 0, r.T}, blockIdx.x, red, [](int row) { return row; });
        return;
    }
    const int block = blockIdx.x - shared.blocks - 1;
    const bool writer = block < 0;
    select_tokens<NW, MAXT>(r.partial, r.bias, r.T, r.nseg, r.E, r.k, s_mask, [&](int t, int32_t sel, float val) {
        if (!writer) return;
        const float g = gate_of(val, r.k);
        if (lane < r.k) {
            r.topk_idx[t * r.k + lane] = sel;
            r.gates[t * r.k + lane] = g;
            s_sel[t][lane] = (uint8_t)sel;
        }
    });
    __syncthreads();
    // lane = expert: its tokens as bits, its rows
    uint32_t tokens = 0;
    for (int t = 0; t < r.T; ++t) tokens |= (uint32_t)((s_mask[t] >> lane) & 1) << t;
    const int count = __popc(tokens);
    const int offset = wave_inclusive_sum(count) - count;
    if (writer) {
        if (threadIdx.x < 64) {
            s_off[lane] = offset;
            if (lane < r.E) {
                r.counts[lane] = count;
                r.offsets[lane] = offset;
            }
            if (lane == 63) r.offsets[r.E] = offset + count;
        }
        __syncthreads();
        for (int a = threadIdx.x; a < r.T * r.k; a += NW * 64) {
            const int t = a / r.k, e = s_sel[t][a - t * r.k];
            int at = s_off[e];
            for (int q = 0; q < t; ++q) at += (int)((s_mask[q] >> e) & 1);
            r.perm[at] = a;
            r.inv_perm[a] = at;
            r.row_token[at] = t;
        }
        return;
    }
    const int units = routed.features >> 4;
    const uint64_t used = __ballot(count > 0);
    const int rank = __popcll(used & ((1ull << lane) - 1));          // place of this expert among those with rows
    const int items = __popcll(used) * units;
    for (int item = block; item < items; item += routed.blocks) {
        const int tile = item / units;
        const int e = __builtin_ctzll(__ballot(count > 0 && rank == tile));
        const uint32_t tok = (uint32_t)__builtin_amdgcn_readlane((int)tokens, e);
        stream_unit_of<true, NW, 1, kSelectStreamRegs>(routed, TileInfo{e, __builtin_amdgcn_readlane(offset, e), __builtin_amdgcn_readlane(count, e)},
                                 item - tile * units, red, [&](int row) {
            int src = 0;
#pragma unroll
            for (int t = 0, c = 0; t < MAXT; ++t)
                if ((tok >> t) & 1) { src = c == row ? t : src; ++c; }
            return src;
        });
    }
}

hipError_t launch_select_gateup(const RoutingArgs& r, const FfnArgs& a, const FfnArgs* shared, hipStream_t s) {
    if (!a.is_bf16 || !a.streaming || r.T > kSelectMaxT || (shared != nullptr && !shared->streaming)) return hipErrorInvalidValue;
    const int64_t units = (int64_t)(a.features / 16) * a.max_tiles, shared_units = shared ? shared->features / 16 : 0;
    const FfnJob jr = make_job(a, (int)(units < kSelectBlocks ? units : kSelectBlocks));
    const FfnJob js = shared ? make_job(*shared, (int)shared_units) : FfnJob{};
    const SelectArgs sel{r.partial, r.bias, r.T, r.d / kRouterSegment, r.E, r.k, r.topk_idx, r.counts, r.offsets, r.perm, r.inv_perm,
                         r.row_token, r.gates};
    const dim3 grid((unsigned)(jr.blocks + js.blocks + 1));
    const bool few = r.T <= 8;
    if (stream_launch_waves(a, shared) == 8) {
        if (few) hipLaunchKernelGGL((select_gateup_kernel<8, 8>), grid, dim3(512), 0, s, jr, js, sel);
        else hipLaunchKernelGGL((select_gateup_kernel<8, 16>), grid, dim3(512), 0, s, jr, js, sel);
    } else {
        if (few) hipLaunchKernelGGL((select_gateup_kernel<4, 8>), grid, dim3(256), 0, s, jr, js, sel);
        else hipLaunchKernelGGL((select_gateup_kernel<4, 16>), grid, dim3(256), 0, s, jr, js, sel);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------
// fp32 layers: every output is ONE chain of fp32 fused multiply-adds over K, ascending, starting at +0 -- kept as such, so
// that the rounding of a chained stack of fp32 layers (where a router may turn a last bit into another expert) does not
// depend on how the work is dealt out.  v_mfma_f32_4x4x1_16b_f32 takes one element of the reduction per instruction, for
// four token rows (broadcast) and 64 features (lane = feature): a wave owns 4 rows x 64 features, a workgroup 16 rows of a
// tile, which is as high (more rows in a workgroup were walked one after the other).  fp32 is used at test scale (d 128, F 256,
// 64 tokens, two experts each), where a launch is bound by round trips to memory: weights are requested a block of 32 elements ahead, x
// a step of 64, the first weights before the rows' numbers are known (against tiles of 160 rows and x requested when needed: 4
// layers of d 384, F 384, 16 experts, 128 tokens, k = 4 203 -> 123 us; 2 of d 256, 1000 tokens 220 -> 139).  Weights 64 elements ahead take twice the registers (one wave
// per SIMD) and more loads than the counter of loads in flight holds: 2 % more over 70 random layers, at worst 8 % (14 tokens, 3
// experts of d 384, F 384: 27.2 -> 29.3 us; that test-scale layer 22.3 -> 23.2).  Cutting K over the waves is faster, but not the same sum.
// ---------------------------------------------------------------------------------------------------------
// The chains of four rows (lane % 4) and 64 features (lane) over K: wp are the lane's weights of the NM matrices, a lane's feature being row
// lane % 16 of 16-row slab lane / 16 (its 32 elements of a K block are four runs of 8, 128 floats apart); `x_row()` gives the lane's row.
template <int NM, typename XRow>
__device__ __forceinline__ void f32_chains(const float* const (&wp)[NM], int K, f32x4_t (&acc)[NM], XRow x_row) {
    const int lane = threadIdx.x & 63;
    struct Block { f32x4_t v[NM][4][2]; };               // 32 elements of the reduction: weights of the lane's feature
    auto fetch_w = [&](Block& b, int kb) {
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) b.v[m][q][h] = *(const f32x4_t*)(wp[m] + (size_t)kb * 512 + q * 128 + 4 * h);
    };
    Block w[2];
    fetch_w(w[0], 0);
    __builtin_amdgcn_sched_barrier(0);                   // (in front of the wait for the row's number)
    const float* xp = x_row() + ((lane >> 2) & 7) * 8;   // octet (lane / 4) % 8 of 64 elements
    f32x4_t x[2][2];                                     // of 64 elements, and of the next 64
    auto fetch_x = [&](f32x4_t (&v)[2], int k0) {
        v[0] = *(const f32x4_t*)(xp + k0);
        v[1] = *(const f32x4_t*)(xp + k0 + 4);
    };
    fetch_x(x[0], 0);
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    auto octet = [&](const Block& b, const f32x4_t (&xv)[2], auto o) {
        constexpr int O = decltype(o)::value;
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int m = 0; m < NM; ++m)
                acc[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[e >> 2][e & 3], b.v[m][O & 3][e >> 2][e & 3], acc[m], 4, O, 0);
    };
    auto step = [&](const f32x4_t (&now)[2], f32x4_t (&next)[2], int k0) {
        fetch_w(w[1], (k0 >> 5) + 1);
        fetch_x(next, min(k0 + 64, K - 64));             // (the last ones are not used)
        __builtin_amdgcn_sched_barrier(0);               // the next block's loads in front of this one's chain
        octet(w[0], now, IntTag<0>{}); octet(w[0], now, IntTag<1>{}); octet(w[0], now, IntTag<2>{}); octet(w[0], now, IntTag<3>{});
        fetch_w(w[0], min((k0 >> 5) + 2, (K >> 5) - 1));
        __builtin_amdgcn_sched_barrier(0);
        octet(w[1], now, IntTag<4>{}); octet(w[1], now, IntTag<5>{}); octet(w[1], now, IntTag<6>{}); octet(w[1], now, IntTag<7>{});
    };
    int k0 = 0;
    for (; k0 + 128 <= K; k0 += 128) {
        step(x[0], x[1], k0);
        step(x[1], x[0], k0 + 64);
    }
    if (k0 < K) step(x[0], x[1], k0);
}
// A lane's weights of `column` of 64 features in packed matrix `e` of [features][K].
__device__ __forceinline__ const float* f32_lane_weights(const float* w, int e, int features, int column, int K) {
    const int lane = threadIdx.x & 63;
    return w + ((size_t)e * (features >> 4) + column * 4 + (lane >> 4)) * ((size_t)K * 16) + (lane & 15) * 8;
}

template <bool GATEUP>
__global__ void __launch_bounds__(256)
ffn_f32_kernel(FfnJob routed, FfnJob shared) {
    int block = blockIdx.y * gridDim.x + blockIdx.x;     // (those past the last find no tile)
    const FfnJob j = pick_job(routed, shared, block);
    const int K = j.K, features = j.features;
    const int column = block % (features >> 6);          // 64 features each
    TileInfo ti;
    if (!fetch_tile<GATEUP ? 0 : 1>(j, block / (features >> 6), ti)) return;
    const int32_t* row_token = j.row_token;
    float* out = (float*)j.out;
    constexpr int NM = GATEUP ? 2 : 1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float* wp[NM] = {f32_lane_weights((const float*)j.w0, ti.expert, features, column, K)};
    if constexpr (GATEUP) wp[1] = f32_lane_weights((const float*)j.w1, ti.expert, features, column, K);
    for (int r0 = wave * 4; r0 < ti.rows; r0 += 16) {   // (no barrier in this kernel)
        const int rr = min(r0 + (lane & 3), ti.rows - 1);   // rows past the tile's end re-read its last row; never stored
        const int src_row = row_token ? row_token[ti.row0 + rr] : ti.row0 + rr;
        f32x4_t acc[NM];
        f32_chains<NM>(wp, K, acc, [&]() { return (const float*)j.in + (size_t)src_row * K; });
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (r0 + i < ti.rows) {
                float v = acc[0][i];
                if (GATEUP) v = silu(v) * acc[NM - 1][i];
                out[(size_t)(ti.row0 + r0 + i) * features + column * 64 + lane] = v;
            }
        }
    }
}

// Down projection and combine of a small fp32 call in one launch (f32_down_combine_fits): a workgroup has 64 features of one token, a wave one of
// its slots at a time (the shared expert is the last), so nothing of the permutation is needed but the slot's row.  A slot's row is the
// same chain as in ffn_f32_kernel (its four rows are one here), the sum over slots combine_kernel's: same bits.  Bound by one chain of
// multiply-adds and two round trips in front of it (64 tokens, k 2, d 128, F 256: 4.8 us against 6.2 and 3.0 in two launches).
template <bool Y_BF16>
__global__ void __launch_bounds__(1024)
down_combine_f32_kernel(DownCombineArgs a) {
    __shared__ float s_row[kF32FusedMaxSlots][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int columns = a.d >> 6;
    const int t = blockIdx.x / columns, column = blockIdx.x - t * columns;
    const int slots = a.k + (a.act_shared != nullptr ? 1 : 0);
    for (int s = wave; s < slots; s += waves) {
        const bool routed = s < a.k;
        const int K = routed ? a.F : a.F_shared;
        const int e = routed ? a.topk_idx[t * a.k + s] : 0, row = routed ? a.inv_perm[t * a.k + s] : t;
        const float* wp[1] = {f32_lane_weights((const float*)(routed ? a.w_down : a.ws_down), e, a.d, column, K)};
        f32x4_t acc[1];
        f32_chains<1>(wp, K, acc, [&]() { return (const float*)(routed ? a.act : a.act_shared) + (size_t)row * K; });
        s_row[s][lane] = acc[0][0];
    }
    __syncthreads();
    if (wave != 0) return;
    float o = 0.0f;
    for (int s = 0; s < a.k; ++s) o = __builtin_fmaf(a.gates[t * a.k + s], s_row[s][lane], o);
    if (a.act_shared != nullptr) o = __builtin_fmaf(1.0f, s_row[a.k][lane], o);
    const size_t at = (size_t)t * a.d + column * 64 + lane;
    if (Y_BF16) ((bf16_t*)a.y)[at] = f32_to_bf16(o);
    else ((float*)a.y)[at] = o;
}

hipError_t launch_down_combine_f32(const DownCombineArgs& a, hipStream_t s) {
    const int slots = a.k + (a.act_shared != nullptr ? 1 : 0);
    if (a.T < 1 || slots > kF32FusedMaxSlots || a.d % 64 != 0 || a.F % 64 != 0 || (a.act_shared != nullptr && a.F_shared % 64 != 0)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)a.T * (unsigned)(a.d / 64)), block((slots < 16 ? slots : 16) * 64);
    if (a.y_bf16) hipLaunchKernelGGL(down_combine_f32_kernel<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(down_combine_f32_kernel<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

template <bool GATEUP>
static hipError_t launch_stream(const FfnArgs& a, const FfnArgs* shared, hipStream_t s) {
    const int width = a.is_bf16 ? 16 : 64;               // output features of a workgroup
    auto job = [&](const FfnArgs* f) {
        return f ? make_job(*f, round_to_xcds((long long)(f->features / width) * f->max_tiles)) : FfnJob{};
    };
    const FfnJob jr = job(&a), js = job(shared);
    if (jr.blocks + js.blocks <= 0) return hipSuccess;
    const dim3 grid((unsigned)(jr.blocks + js.blocks));
    if (!a.is_bf16) {
        // tiles of 16 rows: 262143 tokens, d 4096, k = 17 have 17.8 million workgroups, and a dimension of a grid holds fewer than 2^32 threads
        constexpr unsigned row = 1u << 20;
        const dim3 rows(grid.x < row ? grid.x : row, (grid.x + row - 1) / row);
        hipLaunchKernelGGL(ffn_f32_kernel<GATEUP>, rows, dim3(256), 0, s, jr, js);
    } else {
        auto launch = [&](auto nw) {
            constexpr int NW = decltype(nw)::value;
            if (shared) hipLaunchKernelGGL((ffn_stream_kernel<GATEUP, NW, true>), grid, dim3(NW * 64), 0, s, jr, js);
            else hipLaunchKernelGGL((ffn_stream_kernel<GATEUP, NW, false>), dim3(a.features / 16, a.max_tiles), dim3(NW * 64), 0, s, jr, js);
        };
        if (stream_launch_waves(a, shared) == 8) launch(IntTag<8>{});
        else launch(IntTag<4>{});
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------
// down_combine_kernel: for a handful of tokens the down projection's output rows (T*k x d fp32) are so small that
// writing them out and launching a second kernel to weight and add them costs more than the projection itself.  Here
// a workgroup owns 8 output features of ALL rows, the shared expert's included: the experts that have rows (one
// tile each: an expert holds at most T <= 8 rows) and the shared expert lie one after the other in ONE list of reduction steps,
// which is dealt out evenly over the waves, whatever the number of experts.  A wave adds up each expert's part of its share and
// leaves it in LDS; the parts are added in list order, then y[t] = sum_s g[t][s] * row(t, s) in slot order, plus the
// shared expert's row, exactly as the combine kernel does.  Fixed orders throughout: same bits on every run.
// Eight features and eight rows fill a quarter of a 16 x 16 MFMA, so one instruction takes two K blocks at once: rows 0..7 of A
// and columns 0..7 of B hold the even block, 8..15 the odd one (the two other quarters are not used).  That makes d / 8
// workgroups: every CU of the chip streams at d = 2048, where 16 features each left half of them idle, and with 22 steps (a load of
// weights and one of rows each) in flight a wave's share is one or two round trips.  Wider layers fill the chip with 16 features each, whose blocks are read whole.
// Against 16 features each, passes over the experts and the shared expert's down GEMM in a launch of its own, when it was made
// (whole calls of 8 layers, us): one token, d 2048, F 1408, shared 2816, k 2 to 6 349 -> 306; k = 8, F 1024, no shared expert 303 -> 282;
// 8 tokens, k = 6, shared 784 -> 643; one expert for one token 144 -> 146; d 4096, F 14336, k = 2 1135 -> 1143.  With the short chains
// below one token, k = 8, F 1024 257, 8 tokens, k = 8 810, d 4096, F 14336, one expert, 4 layers 306.
// ---------------------------------------------------------------------------------------------------------
// HALF: 8 features and steps of 64 elements, else 16 features and steps of 32.
template <bool Y_BF16, bool HALF>
__global__ void __launch_bounds__(HALF ? 512 : 1024)
down_combine_kernel(const bf16_t* __restrict__ act, const bf16_t* __restrict__ w_down, int K, int d,
                    const int32_t* __restrict__ sched, const int32_t* __restrict__ counts, int E, const int32_t* __restrict__ inv_perm,
                    const float* __restrict__ gates, const bf16_t* __restrict__ act_shared, const bf16_t* __restrict__ ws_down,
                    int K_shared, int T, int k, void* __restrict__ y) {
    constexpr int NW = HALF ? 8 : 16, UMAX = HALF ? 22 : 11;     // waves; steps in flight per wave
    constexpr int SK = HALF ? 64 : 32, NQ = HALF ? 2 : 4;        // elements of a step; quads of features
    // the parts of (wave, expert), at wave + the expert's place in the list; by (K block parity,) quad of features and row
    __shared__ __attribute__((aligned(16))) f32x4_t red[NW + kFusedDownMaxRows][4][8];
    __shared__ __attribute__((aligned(16))) f32x4_t ys[kFusedDownMaxRows + kFusedDownMaxT][NQ];   // row -> the features
    __shared__ int32_t s_row0[kFusedDownMaxRows], s_rows[kFusedDownMaxRows], s_perm[kFusedDownMaxRows];
    __shared__ float s_gate[kFusedDownMaxRows];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kq = lane >> 4, l8 = lane & 7, par = (lane >> 3) & 1;
    // (the two halves of a unit of 16 features go to the same XCD)
    const int half = HALF ? (blockIdx.x / kXcds) & 1 : 0;
    const int unit = HALF ? blockIdx.x / (2 * kXcds) * kXcds + blockIdx.x % kXcds : blockIdx.x;
    const int f0 = unit * 16 + half * 8;
    // an expert with rows has one tile
    int e_off, e_cnt, e_end;
    if (sched == nullptr) {
        expert_table(counts, E, e_cnt, e_off, e_end);
    } else {
        e_off = sched[kSchedOff + lane]; e_cnt = sched[kSchedCount + lane];
        e_end = sched[kSchedTiles + 64 + lane];
    }
    const int ntiles = __builtin_amdgcn_readlane(e_end, 63);
    if (wave == 0 && e_cnt > 0) {
        s_row0[e_end - 1] = e_off;
        s_rows[e_end - 1] = e_cnt;
    }
    if (wave == 1 && lane < T * k) {                             // (at most 64 assignments)
        s_perm[lane] = inv_perm[lane];
        s_gate[lane] = gates[lane];
    }
    // the list: ntiles experts of `nd` steps, then the shared expert's `ns`
    const int nd = K / SK, ns = act_shared != nullptr ? K_shared / SK : 0;
    const int ntot = ntiles + (ns > 0 ? 1 : 0);
    const int total = ntiles * nd + ns;
    const int lo = wave * total / NW, hi = (wave + 1) * total / NW;   // this wave's share
    // where a lane reads in a step: in the block (two blocks) of 16 rows x 32 K of the weights, in the elements of a row
    const uint32_t a_lane = HALF ? par * 1024 + kq * 256 + (half * 8 + l8) * 16 : lane * 16;
    const uint32_t b_lane = HALF ? par * 64 + kq * 16 : kq * 16;

    int tile = min(lo / nd, ntiles), r = lo - tile * nd;         // (wave-uniform) where the wave is: expert and its step
    struct Part {                                                // what is left of an expert in this wave's share
        const char *a, *b;
        uint32_t b_off;
        int n, at;                                               // steps, place in the list
    };
    auto part = [&](int left) {
        Part p;
        const bool routed = tile < ntiles;
        const int expert = __builtin_amdgcn_readfirstlane(__popcll(__ballot(e_end <= tile))) & 63;   // (64 past the last tile)
        const int row0 = routed ? __builtin_amdgcn_readlane(e_off, expert) : 0;
        const int rows = routed ? __builtin_amdgcn_readlane(e_cnt, expert) : T;
        const int Kt = routed ? K : K_shared;
        const char* w = routed ? (const char*)w_down + (size_t)expert * d * ((size_t)K * 2) : (const char*)ws_down;
        p.a = w + (size_t)unit * ((size_t)Kt * 32) + (size_t)r * (SK * 32);
        p.b = (routed ? (const char*)act : (const char*)act_shared) + (size_t)r * (SK * 2);
        // (rows past the expert's end re-read its last row; their results are never used)
        p.b_off = (uint32_t)(row0 + min(l8, rows - 1)) * (uint32_t)(Kt * 2) + b_lane;
        p.n = min((routed ? nd : ns) - r, left);
        p.at = tile;
        return p;
    };
    auto advance = [&](int n) {                                  // past n steps of the present expert
        r += n;
        if (r == (tile < ntiles ? nd : ns)) {
            r = 0;
            ++tile;
        }
    };
    // Short chains, so that the fp32 rounding is that of a sum in eight parts or less: the steps of a batch go to NA accumulators in
    // turn, the batches are added up.  Error against 64 bits with the intermediate known exactly, 8 tokens, k 6, F 1408, shared 2816:
    // 0.93e-7 (two accumulators 1.12e-7, one chain through the whole share 2.20e-7, every GEMM in eight parts 1.30e-7); d 4096, F 14336,
    // k 2: 1.1e-7 (1.2, 4.7, 5.4).  Four are no slower than one: 8 layers, 8 tokens, k 6, shared 2816 975 -> 960 us.
    constexpr int NA = 4;
    const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4_t acc[NA] = {zero, zero, zero, zero}, sum = zero;
    auto add_up = [&]() {
        sum = sum + ((acc[0] + acc[1]) + (acc[2] + acc[3]));
#pragma unroll
        for (int i = 0; i < NA; ++i) acc[i] = zero;
    };
    auto flush = [&](int at) {                                   // this wave's part of the expert at place `at` is complete
        add_up();
        // (HALF: lanes with bit 3 set hold the odd block, in rows 8..15; else they hold no row)
        if (par == (HALF ? kq >> 1 : 0)) red[wave + at][kq][l8] = sum;
        sum = zero;
    };
    // The first n <= U steps of p and of q behind it, all their loads in flight together.
    auto batch = [&](const Part& p, const Part& q, int n, auto u_tag) {
        constexpr int U = decltype(u_tag)::value;
        bf16x8_t a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = min(u, n - 1);                         // (past the end the last step is fetched again, unused)
            const bool second = v >= p.n;
            const int i = second ? v - p.n : v;
            a[u] = *(const bf16x8_t*)((second ? q.a : p.a) + (size_t)i * (SK * 32) + a_lane);
            b[u] = *(const bf16x8_t*)((second ? q.b : p.b) + (size_t)i * (SK * 2) + (second ? q.b_off : p.b_off));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u < n) {
                if (u == p.n) flush(p.at);
                acc[u % NA] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[u], acc[u % NA], 0, 0, 0);
            }
        }
    };
    for (int s = lo; s < hi;) {
        const Part p = part(hi - s);
        Part q = p;
        int n = p.n;
        if (n < UMAX) {
            advance(p.n);
            if (s + p.n < hi) {
                q = part(hi - s - p.n);
                n = min(p.n + q.n, UMAX);
                advance(n - p.n);
            }
        } else {
            n = UMAX;
            advance(n);
        }
        if (UMAX > 16 && n > 16) batch(p, q, n, IntTag<UMAX>{});
        else if (UMAX > 11 && n > 11) batch(p, q, n, IntTag<(UMAX > 11 ? 16 : 1)>{});
        else if (n > 6) batch(p, q, n, IntTag<11>{});
        else if (n > 3) batch(p, q, n, IntTag<6>{});
        else if (n > 1) batch(p, q, n, IntTag<3>{});
        else batch(p, q, n, IntTag<1>{});
        s += n;
        const int at = n > p.n ? q.at : p.at;
        if (s == hi || at != tile) flush(at);
        else add_up();
    }
    __syncthreads();
    // add the parts of every expert: thread (place in the list, row, quad)
    for (int i = tid; i < ntot * 8 * NQ; i += NW * 64) {
        const int at = i / (8 * NQ), row = i / NQ & 7, q = i % NQ;
        const int first = at * nd, last = at < ntiles ? first + nd : total;
        // the waves whose share holds its first and its last step
        const int w0 = (NW * (first + 1) - 1) / total, w1 = (NW * last - 1) / total;
        f32x4_t v = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int w = w0; w <= w1; ++w)
            if (w * total / NW < (w + 1) * total / NW) {         // (fewer steps than waves leave some without any)
                v = v + red[w + at][q][row];
                if (HALF) v = v + red[w + at][2 + q % 2][row];
            }
        if (at == ntiles) ys[kFusedDownMaxRows + row][q] = v;
        else if (row < s_rows[at]) ys[s_row0[at] + row][q] = v;
    }
    __syncthreads();

    // combine: thread (t, q) owns features f0 + 4*q + 0..3 of token t
    if (tid >= T * NQ) return;
    const int ct = tid / NQ, cq = tid % NQ;
    f32x4_t o = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s = 0; s < k; ++s) {   // slot order = rank order
        const float g = s_gate[ct * k + s];
        const f32x4_t v = ys[s_perm[ct * k + s]][cq];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __builtin_fmaf(g, v[i], o[i]);
    }
    if (act_shared != nullptr) {
        const f32x4_t v = ys[kFusedDownMaxRows + ct][cq];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __builtin_fmaf(1.0f, v[i], o[i]);
    }
    const size_t cidx = (size_t)ct * d + f0 + cq * 4;
    if (Y_BF16) {
        u32x2_t pk;
        pk[0] = pack_bf16x2(o[0], o[1]);
        pk[1] = pack_bf16x2(o[2], o[3]);
        *(u32x2_t*)((bf16_t*)y + cidx) = pk;
    } else {
        *(f32x4_t*)((float*)y + cidx) = o;
    }
}

hipError_t launch_down_combine(const DownCombineArgs& a, hipStream_t s) {
    if (a.T < 1 || a.T > kFusedDownMaxT || a.T * a.k > kFusedDownMaxRows || a.d % 128 != 0 || a.F % 64 != 0 ||
        (a.act_shared != nullptr && a.F_shared % 64 != 0))
        return hipErrorInvalidValue;
    const int features = down_combine_features(a.d);
    const bool half = features == 8;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(a.d / features), dim3(features * 64), 0, s, (const bf16_t*)a.act, (const bf16_t*)a.w_down,
                           a.F, a.d, a.sched, a.counts, a.E, a.inv_perm, a.gates, (const bf16_t*)a.act_shared, (const bf16_t*)a.ws_down, a.F_shared, a.T,
                           a.k, a.y);
    };
    if (a.y_bf16) { if (half) launch(down_combine_kernel<true, true>); else launch(down_combine_kernel<true, false>); }
    else          { if (half) launch(down_combine_kernel<false, true>); else launch(down_combine_kernel<false, false>); }
    return hipGetLastError();
}

hipError_t launch_gateup_stream(const FfnArgs& a, const FfnArgs* shared, hipStream_t s) { return launch_stream<true>(a, shared, s); }
hipError_t launch_down_stream(const FfnArgs& a, const FfnArgs* shared, hipStream_t s) { return launch_stream<false>(a, shared, s); }

}  // namespace lexi
