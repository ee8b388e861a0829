// Expert FFN kernels: grouped gate/up GEMM with fused SwiGLU, grouped down GEMM (paper Sec. 2: E_i(x), the part
// that holds nearly all parameters and FLOPs).  bf16 operands on MFMA with fp32 accumulation.  (fp32 layers take
// the weight-streaming schedule's kernel at every size.)
//
// Orientation: the weight block is the MFMA "A" operand (its 16 rows are features), the token block is the "B"
// operand (its 16 columns are tokens).  In the 16x16 accumulator a lane then owns ONE token (column lane%16) and
// 4 consecutive features (rows 4*(lane/16) + 0..3), so the epilogue writes 8- or 16-byte runs along the feature
// axis, and SwiGLU pairs the gate and up accumulators register by register.
#include "ffn_common.hpp"

namespace lexi {

// ---------------------------------------------------------------------------------------------------------
// ffn_mfma_kernel<GATEUP, NW>
//   Workgroup = NW waves; a token tile of up to 160 rows is shared by all waves through LDS; each wave owns
//   its own 64 weight rows (4 feature blocks of 16) against all rows of the tile (up to 10 token blocks): up to 40
//   accumulator blocks of 16 x 16 (v_mfma_f32_16x16x32_bf16) in at most 256 registers per lane, two waves per SIMD.  Weight
//   rows are not shared between waves and are stored in the packed layout, so their MFMA operand fragments go straight from
//   global memory to registers as fully coalesced 1 KB wave loads; only the token tile passes through LDS.
//   The loop is bound by the bytes a CU pulls through its vector-memory path (it delivers 31 B/clk, against the 47 B/clk
//   that 256 rows x 128 tokens would need at full matrix rate), so the tile is as tall as the registers allow: 160 tokens
//   instead of 128 take 8 to 14 % off the gate/up launches (64 experts, d 2048, F 1024, 2048 tokens, k = 8: 154 -> 137 us).
//   The tokens of a tall tile (more than 96 rows) go from memory to LDS directly, two K-steps ahead in a ring of three stages (tall_step): no
//   registers, no LDS stores and no wait for them at a step's end.  Against the next step's tile through registers into the other of two
//   buffers, same bits: 8 experts, d 4096, F 14336, 4096 tokens, k = 1 gate/up 817 -> 780 us, down 430 -> 407, k = 2 1510 -> 1485 and
//   866 -> 827; 60 experts, F 1408, shared 5632, 8192 tokens, k = 4 620 -> 605 and 372 -> 364; 64 experts, d 2048, F 1024, 4096 tokens,
//   k = 8 239 -> 237 and 172 -> 169.  (Low tiles gain nothing from it, 256 tokens behind a skewed router lose 3 %.)
//   NW = 4: two workgroups share a CU and one's prologue/epilogue overlaps the other's MFMA loop.
//   NW = 8 (DOWN): one workgroup per CU, a token row is fetched for 512 weight rows instead of 256.  8 experts, d 4096,
//   F 14336, 4096 tokens: 950 -> 780 us (k = 2), 506 -> 400 us (k = 1); 64 experts, F 1024, 2048 tokens, k = 8: 102 -> 88 us.
//   Gate/up launches, whose items are shorter, gained nothing from it (between -6 and +15 %).
//   Low tiles (a launch that reads weights for a few rows) have forms of their own.  Up to 96 rows the first weights are
//   requested before the rows' numbers have arrived.  Up to 64 rows a DOWN wave takes 32 features instead of 64, in 128
//   registers, four workgroups per CU: a CU by itself reads at most 45 GB/s from HBM (22 where all 256 do), so a launch takes as
//   long as the CU with the most bytes, and its few column blocks (d / 256) deal out badly.  K 1408, d 2048: 24 experts 29.4 -> 29.0 us, 40: 51.6 -> 46.4, 48:
//   57.6 -> 52.7, 60: 65.3 -> 66.4; K 896, d 1280, 64 experts: 40.9 -> 36.9.  (GATEUP has four times the items: -6 to +8 %.)
//   GATEUP: a wave's blocks 0,1 are gate rows g0..g0+31 and blocks 2,3 the matching up rows, so the epilogue is
//   silu(gate)*up -> bf16 act[row][f]; a workgroup of four waves covers 128 hidden features.
//   DOWN:   a wave's blocks are 64 consecutive output features; the epilogue stores fp32 out[row][j].  Options: the
//           reduction cut in two halves handled by two workgroups that write two planes of `out` (more, shorter work
//           items when a launch would otherwise leave most CUs idle in its last round; the consumer adds the planes);
//           rows stored at out[scatter[row]] in the caller's dtype (layers with one active expert: no combine pass).
//   MIXED: one of the launch's two jobs takes the weight-streaming schedule instead (a shared expert of up to 64 tokens beside
//   routed GEMMs on tiles): its units of 16 features are workgroups of the same launch.
//   Token rows are gathered through row_token (no permuted copy of X is ever materialised).
//   Waves whose feature range lies past `features` (ragged last workgroup column) only help staging the tokens.
// ---------------------------------------------------------------------------------------------------------
template <int S> struct StageTag { static constexpr int value = S; };

typedef __attribute__((address_space(3))) bf16_t lds_bf16;

// Until at most N of the wave's memory operations are on their way (they complete in order) and its LDS operations are done, then
// until the other waves are there too.
template <int N>
__device__ __forceinline__ void wait_and_meet() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// First of the 8 rows that wave `wave` of the workgroup stages in pass p of SR rows.  (Waves past the tile's TT rows repeat its last 8: all
// waves then have the same number of loads on their way.)
template <int SR, int TT>
__device__ __forceinline__ int staged_row(int p, int wave) { return min(SR * p + wave * 8, TT - 8); }

// One K-step on NTB token blocks of a tall tile: stage `rd` against the wave's weights `w`, which are replaced by the next step's as soon as
// they are used; the tokens of two steps ahead are sent for stage `wr` first.  A stage is TT rows of 128 bytes, 16-byte piece c of row r at place
// c ^ (r % 8), so that the fragment reads (frag0, frag1: the lane's first element in either half of a row) fall on all banks.
// `rd` and `wr` are different stages of one array: restrict tells the compiler, which would else wait for all loads to LDS
// before it reads a fragment.  More than 8 blocks leave too few of the 256 registers for all fragments of a half: two at a time, the next
// pair read while the current one is multiplied.
template <int NTB, int NX, int SR, int TT, int WB, int TB>
__device__ __forceinline__ void tall_step(const lds_bf16* __restrict__ rd, lds_bf16* __restrict__ wr, f32x4_t (&acc)[WB][TB], bf16x8_t (&w)[WB][2],
                                          const char* const (&wbase)[WB], uint32_t wnext, const void* in, const uint32_t (&xoff)[NX],
                                          uint32_t xnext, int frag0, int frag1, int wave) {
    constexpr int GB = NTB > 8 ? 2 : NTB;
    constexpr int NG = (NTB + GB - 1) / GB;
#pragma unroll
    for (int p = 0; p < NX; ++p) load_to_lds(in, xoff[p], xnext, wr + staged_row<SR, TT>(p, wave) * BK);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        bf16x8_t b[2][GB];
        auto read_group = [&](int g) {
#pragma unroll
            for (int u = 0; u < GB; ++u)
                if (GB * g + u < NTB)
                    b[g & 1][u] = *(const __attribute__((address_space(3))) bf16x8_t*)(rd + (GB * g + u) * 16 * BK + (ks ? frag1 : frag0));
        };
        read_group(0);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) read_group(g + 1);
            if (NG > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int fb = 0; fb < WB; ++fb)
#pragma unroll
                for (int u = 0; u < GB; ++u)
                    if (GB * g + u < NTB)
                        acc[fb][GB * g + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[fb][ks], b[g & 1][u], acc[fb][GB * g + u], 0, 0, 0);
        }
#pragma unroll
        for (int fb = 0; fb < WB; ++fb) w[fb][ks] = *(const bf16x8_t*)(wbase[fb] + (wnext + (uint32_t)ks * 1024u));
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <bool GATEUP, int NW, int WB, int TT, bool MIXED>
__global__ void __launch_bounds__(NW * 64, WB == 2 ? 4 : 2)
ffn_mfma_kernel(FfnJob routed, FfnJob shared) {
    constexpr int TB = TT / 16, KS = BK / 32;
    constexpr bool LOW = TT <= kLowTileRows;
    constexpr int WF = GATEUP ? 8 * WB : 16 * WB;    // output features of a wave
    constexpr int CB = NW * WF;                      // of the workgroup
    constexpr int ELD = CB + 8;                      // GATEUP: bf16 elements per row of the staged output tile
    constexpr int STAGES_LDS = LOW ? 2 * TT * LDS_LD : 3 * TT * BK;
    constexpr int TILE_LDS = (GATEUP && TT * ELD > STAGES_LDS) ? TT * ELD : STAGES_LDS;
    constexpr int UNIT_LDS = MIXED ? stream_eight_lds<GATEUP>(4) * (int)(sizeof(f32x4_t) / sizeof(bf16_t)) : 0;
    constexpr int LDS_ELEMS = UNIT_LDS > TILE_LDS ? UNIT_LDS : TILE_LDS;
    __shared__ __attribute__((aligned(128))) bf16_t lds[LDS_ELEMS];

    int block = blockIdx.x;
    const FfnJob j = pick_job(routed, shared, block);
    TileInfo ti;
    if (MIXED && j.streams) {
        static_assert(!MIXED || NW == 4, "");
        const int units = j.features >> 4, tile = block / units;
        if (!fetch_tile<GATEUP ? 0 : 1>(j, tile, ti)) return;
        stream_unit_of<GATEUP, NW, 8, 60>(j, ti, block - tile * units, (f32x4_t*)lds,
                                      [&](int r) { return j.row_token ? j.row_token[ti.row0 + r] : ti.row0 + r; });
        return;
    }
    const int K = j.K, features = j.features;
    const bf16_t *in = (const bf16_t*)j.in, *w0 = (const bf16_t*)j.w0, *w1 = (const bf16_t*)j.w1;
    const int32_t *row_token = j.row_token, *scatter = GATEUP ? nullptr : j.scatter;
    void* out = j.out;
    const int ksplit = GATEUP ? 1 : j.ksplit, out_bf16 = j.out_bf16;
    const size_t plane_stride = j.plane_stride;
    int cb, part;
    if (!fetch_item<GATEUP ? 0 : 1>(block, j.sched, (features + CB - 1) / CB, j.M, j.tile_rows, ksplit, ti, cb, part)) return;
    // (wave-uniform, but their divisions run on the vector unit: back to scalar registers, the loop has no vector ones to spare)
    ti.row0 = __builtin_amdgcn_readfirstlane(ti.row0);
    ti.rows = __builtin_amdgcn_readfirstlane(ti.rows);
    ti.expert = __builtin_amdgcn_readfirstlane(ti.expert);
    cb = __builtin_amdgcn_readfirstlane(cb);
    part = __builtin_amdgcn_readfirstlane(part);
    // DOWN with a split reduction: this workgroup covers K-steps [part * steps / ksplit, (part + 1) * steps / ksplit)
    // and writes plane `part`
    const int steps = K / BK;
    const int kstep0 = GATEUP ? 0 : part * steps / ksplit;
    const int nk = GATEUP ? steps : (part + 1) * steps / ksplit - kstep0;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_f0 = cb * CB + wave * WF;  // first output feature
    const bool active = wave_f0 < features;
    const int l16 = lane & 15, kq = lane >> 4;
    const int koff = kq * 8;

    // ---- weight fragments: feature block fb of this wave is 16 packed rows; one K-step of 32 is one 1 KB block, a
    //      lane reads its 16 bytes at lane*16; successive K-steps are 1 KB apart.  The block-row origins are
    //      wave-uniform and live in scalar registers, the lane part is one 32-bit offset (a packed 16-row slab is
    //      32*K bytes, far below 4 GiB): 64-bit per-lane pointers would push the kernel over its 256 registers.
    const char* abase[WB];
#pragma unroll
    for (int fb = 0; fb < WB; ++fb) {
        int row;
        const bf16_t* base = w0;
        if (GATEUP) {
            row = wave_f0 + 16 * (fb % (WB / 2));
            if (fb >= WB / 2) base = w1;
        } else {
            row = wave_f0 + 16 * fb;
        }
        row = active ? row : 0;
        abase[fb] = (const char*)(base + ((size_t)ti.expert * (features >> 4) + (row >> 4)) * ((size_t)K * 16)) +
                    (size_t)kstep0 * (KS * 1024);
    }
    const uint32_t alane = lane * 16;

    // ---- token tile staging: in pass p this thread takes 16 bytes of row staged_row(p) + lane / 8
    constexpr int SR = NW * 8;                       // token rows staged per pass of the workgroup
    constexpr int XP = (TT + SR - 1) / SR;
    int xrow[XP];                                    // the rows of `in` behind them
#pragma unroll
    for (int p = 0; p < XP; ++p) {
        const int r = min(staged_row<SR, TT>(p, wave) + (lane >> 3), ti.rows - 1);   // rows past the group end re-read its last row; never stored
        xrow[p] = row_token ? row_token[ti.row0 + r] : ti.row0 + r;
    }

    // In the form for low tiles the first weights are requested here, while the rows' numbers and the code of the switch below
    // are still on their way (T 64, 60 experts: 1.5 % of the launch).  The form for tall ones requests them behind the switch:
    // alive across it they spill (72 to 96 bytes of scratch per lane; DOWN at K 1024 to 1408 2 to 5 % slower, GATEUP -1 to +1 %).
    bf16x8_t afirst[WB][KS];
    if constexpr (LOW) {
#pragma unroll
        for (int fb = 0; fb < WB; ++fb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) afirst[fb][ks] = *(const bf16x8_t*)(abase[fb] + (alane + (uint32_t)ks * 1024u));
    }

    f32x4_t acc[WB][TB];
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[a][b][v] = 0.0f;

    // The K loop, specialised on the number of 16-token blocks the tile really holds: nothing is staged, read or multiplied
    // for blocks that would only hold padding.
    // Low tiles: the tile of the next K-step is fetched at the top of a step and stored at its end, the token fragments of a half
    // step are read together.
    auto low_loop = [&](auto ntb_tag) {
        constexpr int NTB = decltype(ntb_tag)::value;
        constexpr int NP = (NTB * 16 + SR - 1) / SR;     // passes of this tile
        bf16x8_t areg[WB][KS];
#pragma unroll
        for (int fb = 0; fb < WB; ++fb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) areg[fb][ks] = afirst[fb][ks];
        __builtin_amdgcn_sched_barrier(0);   // (the weights are on their way before the rows' numbers are waited for)
        // byte offsets from `in` (the launcher rejects inputs of 4 GiB or more)
        uint32_t xoff[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) xoff[p] = (uint32_t)(((size_t)xrow[p] * K + (size_t)kstep0 * BK) * 2) + (tid & 7) * 16;
        auto lds_x = [&](int buf) { return lds + buf * (TT * LDS_LD); };
        u32x4_t xreg[NP];
        auto load_x = [&](int kt) {
#pragma unroll
            for (int p = 0; p < NP; ++p) xreg[p] = *(const u32x4_t*)((const char*)in + (xoff[p] + (uint32_t)kt * (BK * 2)));
        };
        auto store_x = [&](int buf) {
#pragma unroll
            for (int p = 0; p < NP; ++p) *(u32x4_t*)(lds_x(buf) + ((tid >> 3) + SR * p) * LDS_LD + (tid & 7) * 8) = xreg[p];
        };
        load_x(0);
        store_x(0);
        __syncthreads();
        for (int kt = 0; kt < nk; ++kt) {
            const int buf = kt & 1;
            const int kn = min(kt + 1, nk - 1);  // the last stage re-fetches itself: branch-free, in bounds, unused
            load_x(kn);
            __builtin_amdgcn_sched_barrier(0);   // keep the token-tile loads in front: they are consumed after the MFMAs
            // (waves of a ragged last column run the same loop on weight row 0 instead of branching around it)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                bf16x8_t b[NTB];
#pragma unroll
                for (int tb = 0; tb < NTB; ++tb) b[tb] = *(const bf16x8_t*)(lds_x(buf) + (tb * 16 + l16) * LDS_LD + ks * 32 + koff);
#pragma unroll
                for (int fb = 0; fb < WB; ++fb)
#pragma unroll
                    for (int tb = 0; tb < NTB; ++tb)
                        acc[fb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(areg[fb][ks], b[tb], acc[fb][tb], 0, 0, 0);
#pragma unroll
                for (int fb = 0; fb < WB; ++fb) areg[fb][ks] = *(const bf16x8_t*)(abase[fb] + (alane + (uint32_t)(kn * KS + ks) * 1024u));
                __builtin_amdgcn_sched_barrier(0);  // refill each fragment right after its last use, one k-step at a time
            }
            store_x(buf ^ 1);
            __syncthreads();
        }
    };
    // Tall tiles: see tall_step.  A wave's loads in program order: weights of step 0 | tokens 0 | tokens 1 | step 0: tokens 2, weights 1 | step 1:
    // tokens 3, weights 2 | ...  At the end of step kt everything but its own NX + WB * KS loads has to be there, tokens kt + 1 among it.
    auto tall_loop = [&](auto ntb_tag) {
        constexpr int NTB = decltype(ntb_tag)::value;
        constexpr int NX = (NTB * 16 + SR - 1) / SR;     // passes of this tile
        constexpr int STAGE = TT * BK;
        // (a different statement for each number: the compiler would move what they have in common in front of the switch)
        asm volatile("; %0 token blocks" ::"n"(NTB));
        bf16x8_t areg[WB][KS];
#pragma unroll
        for (int fb = 0; fb < WB; ++fb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) areg[fb][ks] = *(const bf16x8_t*)(abase[fb] + (alane + (uint32_t)ks * 1024u));
        asm volatile("" ::: "memory");       // (the weights are on their way before the rows' numbers are waited for)
        // byte offsets from `in` (the launcher rejects inputs of 4 GiB or more); row r of a stage takes piece lane % 8 ^ r % 8 of its row
        uint32_t xoff[NX];
#pragma unroll
        for (int p = 0; p < NX; ++p)
            xoff[p] = (uint32_t)(((size_t)xrow[p] * K + (size_t)kstep0 * BK) * 2) + ((lane & 7) ^ (lane >> 3)) * 16;
        auto stage = [&](int at) { return (lds_bf16*)lds + at; };
        auto load_x = [&](int at, int kt) {
#pragma unroll
            for (int p = 0; p < NX; ++p) load_to_lds(in, xoff[p], (uint32_t)kt * (BK * 2), stage(at) + staged_row<SR, TT>(p, wave) * BK);
        };
        load_x(0, 0);
        asm volatile("" ::: "memory");
        load_x(STAGE, min(1, nk - 1));
        wait_and_meet<NX>();
        const int frag0 = l16 * BK + ((kq ^ (l16 & 7)) << 3), frag1 = frag0 ^ 32;
        int rd = 0, wr = 2 * STAGE;
        for (int kt = 0; kt < nk; ++kt) {
            // (the last steps fetch the last one's again: branch-free, in bounds, unused; waves of a ragged last column run on weight row 0)
            tall_step<NTB, NX, SR, TT>(stage(rd), stage(wr), acc, areg, abase, alane + (uint32_t)min(kt + 1, nk - 1) * (KS * 1024u), in, xoff,
                                       (uint32_t)min(kt + 2, nk - 1) * (BK * 2), frag0, frag1, wave);
            rd = rd == 2 * STAGE ? 0 : rd + STAGE;
            wr = wr == 2 * STAGE ? 0 : wr + STAGE;
            wait_and_meet<NX + WB * KS>();
        }
        wait_and_meet<0>();                  // nothing may be on its way to LDS when it is used again
    };
    auto dispatch = [&](auto... n) {
        const int blocks = (ti.rows + 15) >> 4;
        if constexpr (LOW) (void)((blocks == decltype(n)::value ? (low_loop(n), true) : false) || ...);
        else (void)((blocks == decltype(n)::value ? (tall_loop(n), true) : false) || ...);
    };
    if constexpr (TB == 4) dispatch(StageTag<1>{}, StageTag<2>{}, StageTag<3>{}, StageTag<4>{});
    else if constexpr (TB == 6) dispatch(StageTag<1>{}, StageTag<2>{}, StageTag<3>{}, StageTag<4>{}, StageTag<5>{}, StageTag<6>{});
    else dispatch(StageTag<1>{}, StageTag<2>{}, StageTag<3>{}, StageTag<4>{}, StageTag<5>{}, StageTag<6>{}, StageTag<7>{},
                  StageTag<8>{}, StageTag<9>{}, StageTag<10>{});
    static_assert(TB == 4 || TB == 6 || TB == 10, "a K loop for every number of token blocks");
    // ---- epilogue: in a 16 x 16 accumulator block a lane owns token (lane % 16) and features 4*(lane/16) + 0..3
    if (GATEUP) {
        // The workgroup's tokens x 128 features of silu(gate)*up are transposed through LDS (the token-tile
        // buffers are free now), so that the global stores are whole 256-byte rows instead of 8-byte pieces.
        // Row stride 272 B: the 8-byte writes of a half-wave (16 tokens x 2 lane groups) then fall on 64 distinct banks.
        bf16_t* stage = lds;
        __syncthreads();           // every wave is done reading the token tile
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            if (tb * 16 >= ti.rows) break;
#pragma unroll
            for (int fb = 0; fb < WB / 2; ++fb) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = silu(acc[fb][tb][i]) * acc[fb + WB / 2][tb][i];
                u32x2_t pk;
                pk[0] = pack_bf16x2(v[0], v[1]);
                pk[1] = pack_bf16x2(v[2], v[3]);
                *(u32x2_t*)(&stage[(tb * 16 + l16) * ELD + wave * WF + fb * 16 + kq * 4]) = pk;
            }
        }
        __syncthreads();
        constexpr int CH = CB / 8, RP = NW * 64 / CH;    // 16-byte chunks of a row, rows per pass of the workgroup
        const int ch = tid % CH;
        const int f = cb * CB + ch * 8;                 // first of the chunk's 8 features
        if (f < features) {                             // (ragged last column block: features is a multiple of 64)
#pragma unroll
            for (int p = 0; p < TT / RP; ++p) {
                const int r = tid / CH + RP * p;
                if (r < ti.rows)
                    *(u32x4_t*)((bf16_t*)out + (size_t)(ti.row0 + r) * features + f) = *(const u32x4_t*)(&stage[r * ELD + ch * 8]);
            }
        }
    } else {
        // A lane holds 16 bytes of a block of 16 features x 16 rows, so an instruction would store 16 rows of 64 bytes.  Neighbouring
        // lanes (two rows) trade a block, and it stores 8 rows of 128: a CU stores whole cache lines at 58 GB/s, halves of them at
        // 29 (64 CUs, 17 MB: 7.4 against 12.1 us).  4096 tokens, k 8, d 2048, F 1024: launch 187 -> 177 us; 8192 tokens, k 2, F 1408:
        // 136 -> 131.  (A transpose to 64-byte runs per lane measured slower than either.)
        if (!active) return;
        float* plane = (float*)out + (scatter == nullptr ? (size_t)part * plane_stride : 0);
        const bool odd = lane & 1;
        const int f = wave_f0 + kq * 4 + (odd ? 16 : 0);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            if (tb * 16 >= ti.rows) break;
            const int r = tb * 16 + (l16 & ~1);          // the even row of the pair
            int row_even = ti.row0 + r, row_odd = row_even + 1;
            if (scatter != nullptr) {
                // one active expert per token (gate exactly 1): a row is the layer's output row of its token
                const int own = scatter[ti.row0 + min(tb * 16 + l16, ti.rows - 1)];
                const int other = __builtin_amdgcn_update_dpp(own, own, 0xB1, 0xF, 0xF, false);
                row_even = odd ? other : own;
                row_odd = odd ? own : other;
            }
            const size_t o_even = (size_t)row_even * features + f, o_odd = (size_t)row_odd * features + f;
#pragma unroll
            for (int fb = 0; fb < WB; fb += 2) {
                f32x4_t v_even, v_odd;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float keep = odd ? acc[fb + 1][tb][i] : acc[fb][tb][i];
                    const float send = odd ? acc[fb][tb][i] : acc[fb + 1][tb][i];
                    const float got = dpp_f32<0xB1>(send, send);     // quad_perm [1,0,3,2]
                    v_even[i] = odd ? got : keep;
                    v_odd[i] = odd ? keep : got;
                }
                auto store = [&](size_t o, const f32x4_t& v) {
                    if (scatter != nullptr && out_bf16) {
                        u32x2_t pk;
                        pk[0] = pack_bf16x2(v[0], v[1]);
                        pk[1] = pack_bf16x2(v[2], v[3]);
                        *(u32x2_t*)((bf16_t*)out + o) = pk;
                    } else {
                        *(f32x4_t*)(plane + o) = v;
                    }
                };
                if (r < ti.rows) store(o_even + 16 * fb, v_even);
                if (r + 1 < ti.rows) store(o_odd + 16 * fb, v_odd);
            }
        }
    }
}

// pack_kernel: row-major [n_mat][R][K] -> packed layout, one 16-byte (bf16) or 32-byte (fp32) run per thread.
template <typename VEC>
__global__ void __launch_bounds__(256)
pack_kernel(const VEC* __restrict__ src, VEC* __restrict__ dst, int R, int K, size_t runs_total) {
    const size_t run = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x;  // index of the destination run
    if (run >= runs_total) return;
    const size_t runs_per_mat = (size_t)R * (K >> 3);
    const size_t mat = run / runs_per_mat;
    const size_t in_mat = run % runs_per_mat;
    const int i = (int)(in_mat & 15), q = (int)((in_mat >> 4) & 3);
    const size_t blk = in_mat >> 6;
    const int kb = (int)(blk % (size_t)(K >> 5)), rb = (int)(blk / (size_t)(K >> 5));
    const int r = rb * 16 + i, k = kb * 32 + q * 8;
    dst[run] = src[mat * runs_per_mat + ((size_t)r * K + k) / 8];
}

hipError_t launch_pack(const void* src, void* dst, int64_t n_mat, int R, int K, bool is_bf16, hipStream_t s) {
    const size_t runs = (size_t)n_mat * R * (K >> 3);
    if (runs == 0) return hipSuccess;
    // (a dimension of a grid holds fewer than 2^32 threads: 68 GB of bf16 weights)
    const size_t row = (size_t)1 << 20, n = (runs + 255) / 256;
    const dim3 blocks((unsigned)(n < row ? n : row), (unsigned)((n + row - 1) / row));
    if (is_bf16) {
        hipLaunchKernelGGL(pack_kernel<u32x4_t>, blocks, dim3(256), 0, s, (const u32x4_t*)src, (u32x4_t*)dst, R, K, runs);
    } else {
        typedef __attribute__((ext_vector_type(8))) uint32_t u32x8_t;
        hipLaunchKernelGGL(pack_kernel<u32x8_t>, blocks, dim3(256), 0, s, (const u32x8_t*)src, (u32x8_t*)dst, R, K, runs);
    }
    return hipGetLastError();
}

template <bool GATEUP>
static hipError_t launch_ffn(const FfnArgs& a, const FfnArgs* shared, hipStream_t s) {
    if (shared != nullptr && !ffn_joins(a, *shared)) {
        const hipError_t err = launch_ffn<GATEUP>(*shared, nullptr, s);
        return err != hipSuccess ? err : launch_ffn<GATEUP>(a, nullptr, s);
    }
    for (const FfnArgs* f : {&a, shared}) {
        if (f == nullptr) continue;
        const bool tiles = f->is_bf16 && !f->streaming;
        // split reduction and scattered rows exist on the bf16 tile schedule's DOWN only
        if ((f->ksplit > 1 || f->scatter != nullptr) && (!tiles || GATEUP)) return hipErrorInvalidValue;
        if (f->ksplit > 1 && (f->K / BK < f->ksplit || f->scatter != nullptr)) return hipErrorInvalidValue;
        // input rows are addressed with 32-bit byte offsets
        const size_t in_rows = f->row_token ? (size_t)f->in_rows : (size_t)f->M;
        if (f->is_bf16 && in_rows * (size_t)f->K * 2 >= ((size_t)1 << 32)) return hipErrorInvalidValue;
    }
    if (!a.is_bf16 || (a.streaming && (shared == nullptr || shared->streaming)))
        return GATEUP ? launch_gateup_stream(a, shared, s) : launch_down_stream(a, shared, s);
    const bool mixed = a.streaming || (shared != nullptr && shared->streaming);
    auto launch = [&](auto nw, auto wb, auto tt, auto mix) {
        constexpr int NW = decltype(nw)::value, WB = decltype(wb)::value, CB = NW * WB * (GATEUP ? 8 : 16);
        constexpr bool MIXED = decltype(mix)::value != 0;
        auto job = [&](const FfnArgs* f) {
            if (f == nullptr) return FfnJob{};
            const long long columns = f->streaming ? f->features / 16 : (long long)((f->features + CB - 1) / CB) * (f->ksplit > 1 ? f->ksplit : 1);
            return make_job(*f, round_to_xcds(columns * f->max_tiles));
        };
        const FfnJob jr = job(&a), js = job(shared);
        if (jr.blocks + js.blocks <= 0) return;
        hipLaunchKernelGGL((ffn_mfma_kernel<GATEUP, NW, WB, decltype(tt)::value, MIXED>), dim3((unsigned)(jr.blocks + js.blocks)), dim3(NW * 64), 0, s, jr, js);
    };
    int rows = a.streaming ? 0 : a.tile_rows;            // the tallest tile of the launch
    if (shared != nullptr && !shared->streaming && shared->tile_rows > rows) rows = shared->tile_rows;
    auto with = [&](auto nw, auto wb, auto tt) {
        if (mixed) launch(nw, wb, tt, StageTag<1>{});
        else launch(nw, wb, tt, StageTag<0>{});
    };
    if constexpr (!GATEUP) {
        if (a.wide) launch(StageTag<8>{}, StageTag<4>{}, StageTag<kTileRows>{}, StageTag<0>{});
        else if (rows <= kHalfTileRows) with(StageTag<4>{}, StageTag<2>{}, StageTag<kHalfTileRows>{});
    }
    if (!GATEUP && (a.wide || rows <= kHalfTileRows)) return hipGetLastError();
    if (rows <= kLowTileRows) with(StageTag<4>{}, StageTag<4>{}, StageTag<kLowTileRows>{});
    else with(StageTag<4>{}, StageTag<4>{}, StageTag<kTileRows>{});
    return hipGetLastError();
}

hipError_t launch_gateup(const FfnArgs& a, const FfnArgs* shared, hipStream_t s) { return launch_ffn<true>(a, shared, s); }
hipError_t launch_down(const FfnArgs& a, const FfnArgs* shared, hipStream_t s) { return launch_ffn<false>(a, shared, s); }

}  // namespace lexi
