// Internal launch interface between the C ABI (api.hip) and the kernel translation units.
#pragma once
#include "common.hpp"

namespace lexi {

// Height of the token tiles of the grouped GEMMs (rows a tile holds at most), and the XCDs their work is dealt out to.
constexpr int kTileRows = 160;
constexpr int kLowTileRows = 96, kHalfTileRows = 64;   // up to these heights the tile kernel has forms for low tiles
constexpr int kF32TileRows = 16;      // fp32 layers: what a workgroup takes at a time
constexpr int kXcds = 8;

// Tiles of the two grouped GEMMs of a layer (0: gate/up, 1: down), written by the routing kernels: an expert with n rows
// has ceil(n / tile_rows) of them.  In memory: 64 expert offsets, 64 counts, and per GEMM the 64 inclusive sums of the
// experts' tiles.
struct WorkPlan {
    int tile_rows[2];         // tile height, a multiple of 16, at most kTileRows
};
constexpr int kSchedOff = 0, kSchedCount = 64, kSchedTiles = 128, kSchedInts = 256;

struct RoutingArgs {
    const void* x;            // [T][d]
    bool is_bf16;
    const float* w_router;    // [d][E]
    const float* bias;        // [E] or null
    int T, d, E, k;
    WorkPlan plan;
    float* partial;           // [d/128][T][64] segment partials of the logits, where they go through memory (T <= kSmallRouterMaxT, few
                              // experts above kFineRouterMaxT, or many tokens; between kSmallRouterMaxT and kFineRouterMaxT it may share
                              // memory with blk_hist)
    int32_t* topk_idx;        // [T*k]
    float* gates;             // [T*k]
    int32_t* local_rank;      // [T*k]  rank of the assignment inside its router block, per expert
    int32_t* blk_hist;        // [nblk][64] selections per router block and expert
    int32_t* hist_sums;       // [kHistSums][64] the same per workgroup of the permutation, above kPermuteDirectBlocks blocks
    int32_t* counts;          // [E]
    int32_t* offsets;         // [E+1]
    int32_t* perm;            // [T*k]
    int32_t* inv_perm;        // [T*k]
    int32_t* row_token;       // [T*k]  permuted row -> token
    int32_t* sched;           // [kSchedInts]
};

constexpr int kSelectMaxT = 16;         // T at or below which every workgroup of a streaming gate/up launch selects for itself
constexpr int kFusedTailMaxT = 16;     // T at or below which one workgroup does everything after the segment partials
constexpr int kSmallRouterMaxT = 64;   // T at or below which a wave takes one segment of one token
constexpr int kFineRouterMaxT = 1024;  // T at or below which (down to the line above) router and top-k are one launch
// Router blocks (of 16 tokens) up to which every workgroup of the permutation reads all their histograms, and the workgroups it
// has at most above that.
constexpr int kPermuteDirectBlocks = 512;
constexpr int kHistSums = 512;
hipError_t launch_routing(const RoutingArgs& a, hipStream_t s);
hipError_t launch_router_partials(const RoutingArgs& a, hipStream_t s);   // only its first launch (T <= kSmallRouterMaxT)

// One grouped (or dense) GEMM of the expert FFN.
//   GATE/UP:  act[r][f] = silu(in[tok(r)] . Wg[e][f]) * (in[tok(r)] . Wu[e][f])      K = d, features = F
//   DOWN:     out[r][j] = act[r] . Wd[e][j]                                           K = F, features = d
// rows r are the permuted assignment rows (grouped: work list from the scan) or plain token rows (dense, sched == null:
// one group of M rows, expert 0).
struct FfnArgs {
    bool is_bf16;
    bool streaming;            // few rows per expert: use the weight-streaming (HBM-bound) schedule
    bool chained;              // a block of the chained stack: the streaming schedule sums the reduction in four parts
    const void* in;            // row-major [*][K]
    const int32_t* row_token;  // gather map row -> input row, or null (identity)
    int in_rows;               // rows of `in` when row_token is given (bound of the gather)
    const void* w0;            // gate (GATE/UP) or down weights, [E] packed matrices of [features][K]
    const void* w1;            // up weights or null
    int K;                     // reduction length
    int features;              // F (gate/up) or d (down)
    int M;                     // total rows
    int tile_rows;             // as in the work list (WorkPlan)
    int max_tiles;             // upper bound on the number of token tiles
    const int32_t* sched;      // null = dense
    const int32_t* counts;     // null, or [E] (at most kSelectMaxT tokens, streaming): stands in for sched
    int E;
    void* out;                 // GATE/UP: act [rows][F] (layer dtype);  DOWN: [rows][d] fp32
    // DOWN on the tile schedule only:
    bool wide;                 // workgroups of eight waves (512 output features) instead of four (256)
    int ksplit;                // the reduction is cut in ksplit parts, part p writes plane p of `out`
    size_t plane_stride;       // elements between the planes of `out`
    const int32_t* scatter;    // null, or row -> output row: rows are stored at out[scatter[row]] (ksplit must be 1)
    bool out_bf16;             // with scatter: `out` is bf16 (nearest-even rounding of the fp32 result) instead of fp32
};

// Waves per unit of the weight-streaming schedule (bf16), which is also the number of parts its reduction is summed in: eight
// where a CU gets one workgroup at most (twice the loads in flight) or the reduction is very long; with several workgroups
// per CU four are better.  One token, d 2048: dense gate/up 8.8 -> 7.8 us, dense down (K 2816) 8.4 -> 6.5 us, two experts
// 11.0 -> 10.1 us; 32 tokens, down (K 14336) 170 -> 164 us; but 16 tokens, 64 experts: 47 -> 52 us.
// In the chained stack always four: which side of a bf16 rounding a block's input falls on may send a token to another
// expert further down, so the order of a sum there must not depend on the batch the token is in.
inline int stream_waves(int K, int64_t units, bool chained) { return !chained && (units <= 256 || K >= 8192) ? 8 : 4; }
// Parts a streamed sum is taken in: the waves the GEMM has in a launch of its own.
inline int streamed_parts(const FfnArgs& a) { return stream_waves(a.K, (int64_t)(a.features / 16) * a.max_tiles, a.chained); }
// Waves of a launch of one or two streaming GEMMs: eight only where each takes eight parts (four waves can take eight parts, too).
inline int stream_launch_waves(const FfnArgs& a, const FfnArgs* shared) {
    return streamed_parts(a) == 8 && (shared == nullptr || streamed_parts(*shared) == 8) ? 8 : 4;
}

// `shared`: null, or the same GEMM of the layer's shared expert (dense, no scatter).  It goes into the routed one's launch, in front of
// it, where both take the same kind of workgroup (ffn_joins); otherwise it gets a launch of its own.  One launch instead of two: a
// launch costs 4 to 5 us, a second stream 5 to 6 us at its fork and 6 to 10 at its join, and the two fill the last round together.
// Whole calls, us: one token, 8 layers 375 -> 349; 16 tokens, 8 chained layers 726 -> 630; 64 tokens, 6 layers, shared width 5632
// 1293 -> 1282; 256 tokens 1301 -> 1205; 777 tokens, d 1280 852 -> 852; 8192 tokens, 2 layers 1965 -> 1902 (two streams up to 1024
// tokens, one after the other above, each time on the left).  Other sizes against two streams: 9 to 64 tokens 2 to 15 % less, 65
// to 128 tokens, k = 1 (streaming routed experts, tiles of 64 rows) 5 to 15 %; 72 to 1000 tokens with five shapes 0 to 23 % less at 35
// sizes of 40, but 256 tokens, d 4096, 8 experts of F 2048, shared 4096 6 % more, 400 tokens, d 3456, 29 experts 4 %, 600 tokens 2 %: the other
// stream ran the shared gate/up under the routing, and here a few hundred items fall unevenly on the CUs.
inline bool ffn_joins(const FfnArgs& a, const FfnArgs& shared) {
    if (!a.is_bf16 || (a.streaming && shared.streaming)) return true;
    return a.streaming ? !shared.wide : shared.streaming ? !a.wide : a.wide == shared.wide;
}
hipError_t launch_gateup(const FfnArgs& a, const FfnArgs* shared, hipStream_t s);
hipError_t launch_down(const FfnArgs& a, const FfnArgs* shared, hipStream_t s);
// Streaming gate/up of at most kSelectMaxT tokens with the rest of the routing in the same launch: r's router partials are
// there, everything else of it is written.
hipError_t launch_select_gateup(const RoutingArgs& r, const FfnArgs& a, const FfnArgs* shared, hipStream_t s);

// row-major [n_mat][R][K] -> packed expert-weight layout (R % 16 == 0, K % 32 == 0)
hipError_t launch_pack(const void* src, void* dst, int64_t n_mat, int R, int K, bool is_bf16, hipStream_t s);

struct CombineArgs {
    const float* y_slot;       // [T*k][d] fp32, permuted rows; `slot_planes` planes, `slot_plane_stride` elements apart,
                               // that are added (plane order) before the gate is applied
    int slot_planes;
    size_t slot_plane_stride;
    const int32_t* inv_perm;   // [T*k]
    const float* gates;        // [T*k]
    const float* y_shared;     // [T][d] fp32 or null; `shared_planes` planes likewise
    int shared_planes;
    size_t shared_plane_stride;
    const void* x;             // [T][d] layer input (only read for a sigmoid-gated shared expert)
    const void* w_shared_gate; // [d] or null (ungated: coefficient 1)
    bool x_bf16;
    int T, d, k;
    const float* residual;     // [T][d] fp32 added to the result (chained stack), or null; may alias y
    void* y;                   // [T][d]
    bool y_bf16;
    void* u_next;              // chained stack: [T][d] layer dtype, the next block's normalised input, or null
};
hipError_t launch_combine(const CombineArgs& a, hipStream_t s);

// Down projection and combine of a decode-sized batch in one launch (bf16 layers, T <= kFusedDownMaxT, T*k <=
// kFusedDownMaxRows, shared expert absent or ungated): y[t] = sum_s gates[t][s] * (act[row(t, s)] . W_down[e]) in slot
// order, then the shared expert's row, whose down projection is part of the launch.
// Limits: an expert's rows are the 8 columns of half an MFMA operand, all rows' features lie in LDS.  Up to them, against separate
// launches, 4 layers, one to 8 tokens, k 1 to 16, with and without a shared expert: d 2048 7 to 14 % less time, d 4096 5 to 10 %; d 640, whose 80
// workgroups leave most CUs idle, 3 to 15 % less up to 8 assignments, up to 15 % more with 16 to 64 of them.
constexpr int kFusedDownMaxT = 8;
constexpr int kFusedDownMaxRows = 64;
// Output features of a workgroup: 8 where that is at most one workgroup per CU, else 16, with as many waves as features (8 at d 2176
// to 4096, 8 layers, one to 8 tokens: 0 to 10 % more time).
inline int down_combine_features(int d) { return d <= 2048 ? 8 : 16; }
struct DownCombineArgs {
    const void* act;           // [T*k][F] bf16 (fp32 layers: fp32, as the weights and act_shared), permuted rows
    const void* w_down;        // [E] packed matrices of [d][F]
    int F, d, T, k;
    const int32_t* sched;      // work list (one tile per expert with rows), or null: then
    const int32_t* counts;     // [E]
    int E;
    const int32_t* topk_idx;   // [T*k] (fp32 layers only)
    const int32_t* inv_perm;   // [T*k]
    const float* gates;        // [T*k]
    const void* act_shared;    // [T][F_shared] or null: the shared expert, added with coefficient 1
    const void* ws_down;       // packed [d][F_shared]
    int F_shared;
    void* y;                   // [T][d]
    bool y_bf16;
};
hipError_t launch_down_combine(const DownCombineArgs& a, hipStream_t s);
// The same for fp32 layers (topk_idx in place of sched and counts): a workgroup per token and 64 features, and
// every slot pulls its own 256 bytes of weights per element of the reduction, where the tiles of separate launches share them.  Bound by what a
// CU pulls, so the line lies there.  Down + combine, separate launches against one, us (KB per CU): 64 tokens, k 2, d 128, F 256 9.2 / 4.8
// (131); 1024 tokens, d 128, F 64 8.1 / 5.8 (262); 128 tokens, d 256, F 256 8.9 / 6.1 (262); d 384, F 128, shared 128 7.1 / 6.5 (295); then d 384,
// F 384: 8 tokens, k 4 8.1 / 7.1 (393; the call 23.2 / 23.1), 64 tokens, k 2 9.0 / 8.8 (393; 31.4 / 31.7), 128 tokens 10.0 / 10.9 (590), 16 tokens,
// k 8 8.9 / 12.2 (786).
constexpr int kF32FusedMaxSlots = 65;
constexpr int64_t kF32FusedBytesPerCu = 300 << 10;
inline bool f32_down_combine_fits(int T, int k, int d, int F, int F_shared) {
    const int64_t groups = (int64_t)T * (d / 64);
    return (groups + 255) / 256 * ((int64_t)k * F + F_shared) * 256 <= kF32FusedBytesPerCu;
}
hipError_t launch_down_combine_f32(const DownCombineArgs& a, hipStream_t s);

// chained stack: the fp32 hidden state h = widened x, and the first block's normalised MoE input u (layer dtype)
constexpr float kRmsEps = 1e-6f;
hipError_t launch_start_chain(const void* x, bool is_bf16, int T, int d, float eps, float* h, void* u, hipStream_t s);

// Stage-1 profiling: squared-difference reduction over the slot rows of one baseline pass.
constexpr int kProfileMaxK = 64;
struct ProfileKList {          // passed to the kernel by value
    int32_t n;
    int32_t k[kProfileMaxK];
};
struct ProfileArgs {
    const float* y_slot;       // [T*k_base][d] fp32, permuted rows
    const int32_t* inv_perm;   // [T*k_base]
    const float* gates;        // [T*k_base] baseline gates
    int T, d, k_base;
    ProfileKList klist;
    float* part;               // [n][T] per-token squared norms
    float* delta;              // [n]
};
hipError_t launch_profile(const ProfileArgs& a, hipStream_t s);

}  // namespace lexi
