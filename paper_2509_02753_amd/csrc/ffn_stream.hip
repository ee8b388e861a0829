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

namespace lexi {

template <bool GATEUP, int NW>
__global__ void __launch_bounds__(NW * 64)
ffn_stream_kernel(FfnJob routed, FfnJob shared) {
    __shared__ __attribute__((aligned(16))) f32x4_t red[NW][2][64];
    int block = blockIdx.x;
    const FfnJob j = pick_job(routed, shared, block);
    const int units = j.features >> 4;
    const int tile = block / units;
    TileInfo ti;
    if (!fetch_tile<GATEUP ? 0 : 1>(j.sched, tile, j.M, j.tile_rows, ti)) return;
    stream_unit<GATEUP, NW>(j, ti, block - tile * units, red);
}

// ---------------------------------------------------------------------------------------------------------
// fp32 layers: every output is ONE chain of fp32 fused multiply-adds over K, ascending, starting at +0 -- kept as such, so
// that the rounding of a chained stack of fp32 layers (where a router may turn a last bit into another expert) does not
// depend on how the work is dealt out.  v_mfma_f32_4x4x1_16b_f32 takes one element of the reduction per instruction, for
// four token rows (broadcast) and 64 features (lane = feature): a wave owns 4 rows x 64 features, a workgroup 16 rows of a
// tile at a time.  fp32 is used at test scale (d 128, F 256, 64 tokens, two experts each), where a launch is bound by the
// latency of the chain (4.7 ns an instruction): 7.4 + 8.3 us for that layer's two GEMMs, where one output element per thread
// walking K alone took 636 + 664 us (same bits).  Cutting K over the waves is faster still (4.8 + 4.6 us) but not the same sum.
// ---------------------------------------------------------------------------------------------------------
template <bool GATEUP>
__global__ void __launch_bounds__(256)
ffn_f32_kernel(FfnJob routed, FfnJob shared) {
    int block = blockIdx.x;
    const FfnJob j = pick_job(routed, shared, block);
    const int K = j.K, features = j.features;
    const int column = block % (features >> 6);          // 64 features each
    TileInfo ti;
    if (!fetch_tile<GATEUP ? 0 : 1>(j.sched, block / (features >> 6), j.M, j.tile_rows, ti)) return;
    const float *in = (const float*)j.in, *w0 = (const float*)j.w0, *w1 = (const float*)j.w1;
    const int32_t* row_token = j.row_token;
    float* out = (float*)j.out;
    constexpr int NM = GATEUP ? 2 : 1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // packed weights: a lane's feature is row lane % 16 of 16-row slab lane / 16; its 32 elements of a K block are four runs
    // of 8, 128 floats apart
    const size_t slab = (size_t)ti.expert * (features >> 4) + column * 4 + (lane >> 4);
    const float* wp[2] = {w0 + slab * ((size_t)K * 16) + (lane & 15) * 8, GATEUP ? w1 + slab * ((size_t)K * 16) + (lane & 15) * 8 : nullptr};
    struct Block { f32x4_t v[NM][4][2]; };
    auto fetch_w = [&](Block& b, int kb) {
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) b.v[m][q][h] = *(const f32x4_t*)(wp[m] + (size_t)kb * 512 + q * 128 + 4 * h);
    };
    for (int r0 = wave * 4; r0 < ti.rows; r0 += 16) {   // (no barrier in this kernel)
        const int rr = min(r0 + (lane & 3), ti.rows - 1);   // rows past the tile's end re-read its last row; never stored
        const int src_row = row_token ? row_token[ti.row0 + rr] : ti.row0 + rr;
        const float* xp = in + (size_t)src_row * K + ((lane >> 2) & 7) * 8;   // octet (lane / 4) % 8 of 64 elements
        f32x4_t acc[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) acc[m] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        Block w[2];
        fetch_w(w[0], 0);
        for (int k0 = 0; k0 < K; k0 += 64) {            // (K is a multiple of 64)
            const f32x4_t x0 = *(const f32x4_t*)(xp + k0), x1 = *(const f32x4_t*)(xp + k0 + 4);
            auto octet = [&](const Block& b, auto o) {  // elements k0 + 8 * O .. + 7, octet O % 4 of K block O / 4
                constexpr int O = decltype(o)::value;
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int m = 0; m < NM; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(e < 4 ? x0[e & 3] : x1[e & 3], b.v[m][O & 3][e >> 2][e & 3], acc[m], 4, O, 0);
            };
            fetch_w(w[1], (k0 >> 5) + 1);
            __builtin_amdgcn_sched_barrier(0);   // the next block's loads in front of this one's chain
            octet(w[0], IntTag<0>{}); octet(w[0], IntTag<1>{}); octet(w[0], IntTag<2>{}); octet(w[0], IntTag<3>{});
            fetch_w(w[0], min((k0 >> 5) + 2, (K >> 5) - 1));   // (the last one is not used)
            __builtin_amdgcn_sched_barrier(0);
            octet(w[1], IntTag<4>{}); octet(w[1], IntTag<5>{}); octet(w[1], IntTag<6>{}); octet(w[1], IntTag<7>{});
        }
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
        hipLaunchKernelGGL(ffn_f32_kernel<GATEUP>, grid, dim3(256), 0, s, jr, js);
    } else {
        const int64_t units = (int64_t)(a.features / 16) * a.max_tiles + (shared ? (int64_t)(shared->features / 16) * shared->max_tiles : 0);
        const int K = shared && shared->K > a.K ? shared->K : a.K;
        if (stream_waves(K, units, a.chained) == 8) hipLaunchKernelGGL((ffn_stream_kernel<GATEUP, 8>), grid, dim3(512), 0, s, jr, js);
        else hipLaunchKernelGGL((ffn_stream_kernel<GATEUP, 4>), grid, dim3(256), 0, s, jr, js);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------
// down_combine_kernel: for a handful of tokens the down projection's output rows (T*k x d fp32) are so small that
// writing them out and launching a second kernel to weight and add them costs more than the projection itself.  Here
// a workgroup of 16 waves owns 16 output features of ALL rows: it walks the experts that have rows (one tile each:
// an expert holds at most T <= 8 rows), several at a time -- the waves are dealt out as (experts per pass) x (parts
// of the reduction), the fewer experts the finer the split -- adds the parts in order through LDS, keeps the rows'
// 16 features in an LDS table, and finally forms y[t] = sum_s g[t][s] * row(t, s) in slot order, plus the shared
// expert's row, exactly as the combine kernel does.  Fixed orders throughout: same bits on every run.
// ---------------------------------------------------------------------------------------------------------
template <bool Y_BF16>
__global__ void __launch_bounds__(1024)
down_combine_kernel(const bf16_t* __restrict__ act, const bf16_t* __restrict__ w_down, int K, int d,
                    const int32_t* __restrict__ sched, const int32_t* __restrict__ inv_perm,
                    const float* __restrict__ gates, const float* __restrict__ y_shared, int T, int k, void* __restrict__ y) {
    __shared__ __attribute__((aligned(16))) f32x4_t red[16][64];
    __shared__ __attribute__((aligned(16))) f32x4_t ys[kFusedDownMaxRows][4];   // row -> the unit's 16 features

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int unit = blockIdx.x;   // output features 16*unit .. 16*unit+15
    const int nkb = K >> 5;
    // an expert with rows has one tile
    const int e_off = sched[kSchedOff + lane], e_cnt = sched[kSchedCount + lane];
    const int e_end = sched[kSchedTiles + 64 + lane];
    const int ntiles = __builtin_amdgcn_readlane(e_end, 63);
    // combine: thread (t, q) owns features 16*unit + 4*q + 0..3 of token t; what it adds at the end that does not
    // depend on the projection is fetched now, under the weight stream
    const bool combiner = tid < T * 4;
    const int ct = tid >> 2, cq = tid & 3;
    const size_t cidx = (size_t)ct * d + unit * 16 + cq * 4;
    f32x4_t shared_row = {0.0f, 0.0f, 0.0f, 0.0f};
    if (combiner && y_shared != nullptr) shared_row = *(const f32x4_t*)(y_shared + cidx);
    constexpr int KPRE = 8;        // slots whose row index and gate are fetched ahead
    int32_t pre_row[KPRE];
    float pre_gate[KPRE];
#pragma unroll
    for (int s = 0; s < KPRE; ++s) {
        const bool have = combiner && s < k;
        pre_row[s] = have ? inv_perm[(size_t)ct * k + s] : 0;
        pre_gate[s] = have ? gates[(size_t)ct * k + s] : 0.0f;
    }
    // waves per expert: 16 for one expert, ..., 1 for nine or more (then 16 experts per pass)
    const int wpt = ntiles >= 9 ? 1 : ntiles >= 5 ? 2 : ntiles >= 3 ? 4 : ntiles == 2 ? 8 : 16;
    const int per_pass = 16 / wpt;
    const int sub = wave / wpt, kpart = wave - sub * wpt;

    for (int t0 = 0; t0 < ntiles; t0 += per_pass) {
        const int tile = t0 + sub;
        const bool live = tile < ntiles;   // wave-uniform
        int row0 = 0, rows = 0;
        f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
        if (live) {
            const int expert = __builtin_amdgcn_readfirstlane(__popcll(__ballot(e_end <= tile)));
            row0 = __builtin_amdgcn_readlane(e_off, expert);
            rows = min(__builtin_amdgcn_readlane(e_cnt, expert), 16);
            const int kb0 = kpart * nkb / wpt, kb1 = (kpart + 1) * nkb / wpt;
            const bf16_t* a0 = w_down + ((size_t)expert * (d >> 4) + unit) * ((size_t)K * 16) + lane * 8;
            // rows past the expert's end re-read its last row; their results are never used
            const bf16_t* xp = act + (size_t)(row0 + min(l16, rows - 1)) * K + kq * 8;
            auto k_step = [&](int kb) {
                const bf16x8_t ag = *(const bf16x8_t*)(a0 + (size_t)kb * 512);
                const bf16x8_t b = *(const bf16x8_t*)(xp + kb * 32);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ag, b, acc, 0, 0, 0);
            };
            constexpr int UNROLL = 11;   // K blocks whose loads are in flight together
            int kb = kb0;
            for (; kb + UNROLL <= kb1; kb += UNROLL) {
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) k_step(kb + u);
            }
            for (; kb + 4 <= kb1; kb += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) k_step(kb + u);
            }
            for (; kb < kb1; ++kb) k_step(kb);
        }
        red[wave][lane] = acc;
        __syncthreads();
        if (live && kpart == 0) {
            f32x4_t g = red[wave][lane];
            for (int p = 1; p < wpt; ++p) g += red[wave + p][lane];
            if (l16 < rows) ys[row0 + l16][kq] = g;   // lane owns row (lane % 16), features 4*(lane/16) + 0..3
        }
        __syncthreads();
    }

    if (!combiner) return;
    f32x4_t o = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s = 0; s < k; ++s) {   // slot order = rank order
        int32_t row;
        float g;
        if (s < KPRE) {
            row = pre_row[0]; g = pre_gate[0];
#pragma unroll
            for (int i = 1; i < KPRE; ++i)
                if (s == i) { row = pre_row[i]; g = pre_gate[i]; }
        } else {
            row = inv_perm[(size_t)ct * k + s];
            g = gates[(size_t)ct * k + s];
        }
        const f32x4_t v = ys[row][cq];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __builtin_fmaf(g, v[i], o[i]);
    }
    if (y_shared != nullptr) {
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __builtin_fmaf(1.0f, shared_row[i], o[i]);
    }
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
    if (a.T < 1 || a.T > kFusedDownMaxT || a.T * a.k > kFusedDownMaxRows || a.d % 16 != 0 || a.F % 32 != 0)
        return hipErrorInvalidValue;
    const dim3 grid(a.d / 16);
    if (a.y_bf16)
        hipLaunchKernelGGL(down_combine_kernel<true>, grid, dim3(1024), 0, s, (const bf16_t*)a.act, (const bf16_t*)a.w_down,
                           a.F, a.d, a.sched, a.inv_perm, a.gates, a.y_shared, a.T, a.k, a.y);
    else
        hipLaunchKernelGGL(down_combine_kernel<false>, grid, dim3(1024), 0, s, (const bf16_t*)a.act, (const bf16_t*)a.w_down,
                           a.F, a.d, a.sched, a.inv_perm, a.gates, a.y_shared, a.T, a.k, a.y);
    return hipGetLastError();
}

hipError_t launch_gateup_stream(const FfnArgs& a, const FfnArgs* shared, hipStream_t s) { return launch_stream<true>(a, shared, s); }
hipError_t launch_down_stream(const FfnArgs& a, const FfnArgs* shared, hipStream_t s) { return launch_stream<false>(a, shared, s); }

}  // namespace lexi
