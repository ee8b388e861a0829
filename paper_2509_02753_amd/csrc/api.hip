// C ABI of the library: argument validation, workspace slicing and the per-layer launch sequence.
// Nothing here allocates, synchronises or copies to the host; every launch goes to the caller's stream.
#include "../../include/lexi_probe.h"
#include "kernels.hpp"
#include <math.h>
#include <mutex>

namespace {

using namespace lexi;

// (The lines from here to kStreamDenseRows, and the prices of gemm_cost below, were fitted when the streaming loop had one K block in flight
// and tall tiles got their tokens through registers.  Both loops are up to a fifth faster now; the lines have not been measured again.)
constexpr int kStreamRowsPerExpert = 2;   // mean rows per expert at or below which the routed FFN streams weights
// The down projection has few column blocks (d / 256): where the tile schedule would have no more than
// kStreamDownMaxItems work items, it streams up to kStreamDownRowsPerExpert mean rows per expert.  (A unit of the streaming
// schedule reads all of its tile's rows for 16 output features: at 16 rows per expert, d 4096, F 14336 it takes 228 us
// against 161 us on the tile schedule with the reduction cut in two, at 128 rows 1222 against 212 us.)
// With more rows it still streams while its units are few: the tile schedule then is one chain of K-steps on a few CUs (0.4
// us a step), the units read little beside the weights.  Whole call, streaming against tiles: 24 against 36 us (13 rows, 3
// experts, d 640, F 2624), 27 / 32 (48 rows, 3 experts, d 512, F 1408), 60 / 66 (14 rows, 24 experts, d 640, F 2624: 960 units
// of 16 rows), but 58 / 50 (22 rows, 8 experts, d 2560, F 1408: 2560) and 60 / 51 (39 rows, 6 experts, d 1024, F 4096: 3072).  From 64 rows on a wave's chain of
// loads is as long (28 / 28 at 126 rows, 1 expert, d 512, F 896), except where the reduction is short (25 / 31 at 73 rows, F 192).
constexpr int kStreamDownMaxItems = 256;
constexpr int kStreamDownRowsPerExpert = 8;
constexpr int kStreamShortK = 512;
constexpr int kStreamDownUnits = 1024;    // units x their 16-row blocks (x parts the tile schedule would cut the reduction in)
constexpr int kStreamDenseRows = 64;      // token count at or below which the shared expert streams weights

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Launch plan of one GEMM on the tile schedule.  A launch runs (token tiles x column blocks) work items on the chip's
// workgroup slots: 512 of four waves (two per CU, 256 weight rows each) or 256 of eight (one per CU, 512 weight rows: a
// token row is fetched for twice as many weight rows, which is what the loop is bound by, but a partly filled last round
// costs nearly a whole one).  The number of rows an expert gets is only known on the device; here they are taken as spread
// around rows / groups as a balanced router leaves them.
struct TilePlan {
    bool wide;        // eight waves
    int tile_rows;    // tile height
    int ksplit;       // parts of the reduction
};

// Relative duration of a launch on the tile schedule: rounds of the chip times an item's duration (in 16-row blocks x
// K-steps of a four-wave workgroup), the tallest item once.  An item pays about 3 blocks' worth per K-step whatever its height
// (the weight stream) and `store` K-steps' worth per block for storing its rows.  Launches of at most one four-wave item per
// CU are priced apart, at 0.4 of a round: alone on its CU an item is faster than beside another (gate/up, 3315 tokens, k = 1, 8
// experts of d 2560, F 896: 224 items of 128 rows 44 us, 392 of 64 rows 57).  A column block counts as a whole one where only
// part of it holds features.  Fitted on 168 routed launches (60 to 3500 tokens, with and without a router bias, each timed at
// every height in both forms): against 128 rows everywhere the choice takes gate/up launches from +1.3 % (constants without the
// round of single items) to -0.8 %, down launches from -0.2 to -3.4 %, and the worst gate/up launch from 1.36 to 1.16 times.
double gemm_cost(int64_t rows, int groups, int K, int features, int store, const TilePlan& p, int col_width) {
    const double mean = (double)rows / groups, sd = groups > 1 ? sqrt(mean * (1.0 - 1.0 / groups)) : 0.0;
    const double in_use = groups > 1 && mean < 4.0 ? groups * (1.0 - exp(-mean)) : groups;
    double tiles = 0.0, blocks = 0.0, tallest = 0.0;
    for (double z : {-1.28, -0.52, 0.0, 0.52, 1.28}) {     // fifths of a normal distribution
        const double r = fmax(mean + z * sd, 1.0);
        const double n = ceil(r / p.tile_rows), nb = ceil(r / 16.0);
        tiles += n / 5.0;
        blocks += nb / 5.0;
        tallest = fmax(tallest, ceil(nb / n));
    }
    const double height = blocks / tiles;
    const double rounds = tiles * in_use * ((features + col_width - 1) / col_width) * p.ksplit / (p.wide ? 256.0 : 512.0);
    const double full = floor(rounds), part = rounds - full;
    double last = 0.0;                                      // the partly filled last round
    if (p.wide) last = 0.7 + 0.3 * part;
    else if (full == 0.0) last = part <= 0.5 ? 0.4 : 1.0;
    else last = 0.25 + 0.75 * part;
    if (full > 0.0 && part <= 0.02) last = 0.0;
    const double steps = (double)(K / 64) / p.ksplit, scale = p.wide ? 0.86 : 1.0;
    const double item = ((height + (p.wide ? 3.3 : 3.0)) * steps + store * height) * scale;
    return (full + last) * item + (tallest - height) * (steps + store) * scale;
}

// Token tiles of a launch at most, whatever the routing: an expert with n rows has ceil(n / tile_rows) tiles.
inline int64_t max_tiles(int64_t rows, int groups, int tile_rows) { return rows / tile_rows + (rows < groups ? rows : groups); }

// The best height for four-wave workgroups.  With few rows per expert, where the heights are nearly equal for a balanced
// router, a taller tile has to be clearly better: a lower one spreads the rows of a skewed router over more, shorter items
// (batch-256 decode with Zipf-distributed experts: 1305 us at 64 rows, 1399 at 160).
// `gateup`: above 48 rows per expert lower tiles only stream the weights again behind a skewed router, unless a launch has at
// most one of them per CU however the rows fall (1296 tokens, k = 1, 16 experts of d 3328, F 1408: 93 us at 64 rows, 96 at 96,
// 71 at 128; but 190 tokens, k = 4, 6 experts of d 2048, F 896: the whole call 49 us at 64 rows, 61 at 160).
TilePlan plan_narrow_tiles(int64_t rows, int groups, int K, int features, int store, int ksplit, int col_width, bool gateup) {
    TilePlan best{false, 0, ksplit};
    double cost = 0.0;
    for (int h : {64, 96, 128, 160}) {
        const int64_t items = max_tiles(rows, groups, h) * ((features + col_width - 1) / col_width);
        if (gateup && h < 128 && rows > (int64_t)48 * groups && items > 256) continue;
        const TilePlan p{false, h, ksplit};
        const double c = gemm_cost(rows, groups, K, features, store, p, col_width);
        if (best.tile_rows == 0 || c < (rows < (int64_t)48 * groups ? 0.98 : 1.0) * cost) { best = p; cost = c; }
    }
    return best;
}
TilePlan plan_gateup_tiles(int64_t rows, int groups, int K, int features) {
    return plan_narrow_tiles(rows, groups, K, features, 4, 1, 128, true);
}

// The reduction is cut in two where a launch with a long one cannot fill half the slots: twice as many items of half the
// length, whose results land in two planes of the output that the consumer adds.  Eligible: at least 32 K-steps of 64, an
// even number of them.  Taken when the time saved outweighs writing and re-reading the second plane.  (For launches of
// several rounds, e.g. 1100 items of 14336, the split measured no gain in the down GEMM and cost the combine a second
// plane; four parts measured 0 to 10 % slower than two on launches of 72 to 192 items.)
inline bool ksplit_eligible(int K) { return K / 64 >= 32 && (K / 64) % 2 == 0; }
inline bool down_streams(int64_t rows, int groups, int K, int features, bool direct) {
    if (rows <= (int64_t)kStreamDownRowsPerExpert * groups) return true;
    if (direct && K <= kStreamShortK) return false;   // tiles store the layer's output rows: no combine launch
    if (rows > (int64_t)(K <= kStreamShortK ? 128 : 64) * groups) return false;
    const int blocks = rows <= (int64_t)16 * groups ? 1 : rows <= (int64_t)32 * groups ? 2 : rows <= (int64_t)64 * groups ? 4 : 8;
    return (int64_t)(features / 16) * groups * blocks * (ksplit_eligible(K) ? 2 : 1) <= kStreamDownUnits;
}
TilePlan plan_down_tiles(int64_t rows, int groups, int K, int features, bool allow_split, bool direct) {
    constexpr int kPlanRows = 128;
    const double ragged = groups > 1 ? 0.5 * (double)(groups < rows ? groups : rows) : (rows % kPlanRows ? 0.5 : 0.0);
    const double items = ((double)(rows / kPlanRows) + ragged) * ((features + 255) / 256);
    if (allow_split && ksplit_eligible(K) && items <= 256) {
        const double t_item = (2.0 * kPlanRows * 256.0 * K) / 3.9e12;           // one item at what one CU sustains
        const double t_plane = 2.0 * (double)rows * features * 4.0 / 5.0e12;    // second plane: written once, read once
        // (rows stored straight into the layer's output need no combine launch at all while the reduction is whole)
        if (0.5 * t_item > 1.5 * t_plane + (direct ? 20e-6 : 0.0))
            return plan_narrow_tiles(rows, groups, K, features, 7, 2, 256, false);
    }
    TilePlan best = plan_narrow_tiles(rows, groups, K, features, 7, 1, 256, false);
    // The eight-wave form needs a few hundred rows per expert: with fewer a launch streams weights, and a skewed router leaves
    // its few large items unevenly spread (1464 tokens, k = 5, 60 experts, d 1792, F 2240: 148 us behind a biased router
    // against 124 at 128 rows, 123 on both sides behind an unbiased one).
    if (rows < (int64_t)250 * groups) return best;
    double cost = gemm_cost(rows, groups, K, features, 7, best, 256);
    for (int h : {kTileRows, 128}) {
        const TilePlan p{true, h, 1};
        const double c = gemm_cost(rows, groups, K, features, 7, p, 512);
        if (c < cost) { best = p; cost = c; }
    }
    return best;
}

// Tokens up to which the shared expert's GEMMs take the routed GEMMs' kind of workgroup and tile height, so that each shares the
// routed one's launch and form of the kernel (256 tokens: 1268 us at 128 rows, 1222 at the routed GEMMs' 64).  Beside an eight-wave
// routed GEMM 128 rows; beside a streaming one 64 for the down GEMM, whose form has four workgroups per CU instead of two: most of the
// launch are units that stream (100 tokens, k = 1, 64 experts of F 1024, shared 1408, 4 layers: d 4096 1197 us at 128 rows, 1076 at
// 64, two launches in turn 1376; d 2048 637, 592, 763.  Gate/up has two per CU at any height: 128 or 64 rows within 2 %).  With more tokens a
// shared expert fills the chip by itself and keeps the tallest tiles.
constexpr int kSharedJoinsMaxT = 1024;
constexpr int kSharedTileRows = 128;
constexpr int kMaxDevices = 16;

// Scratch of lexi_moe_layer_forward_static: the workspace of one decode-sized layer call, held in the library's own
// device image so that the call needs no allocation and no workspace argument.  Every GPU the library runs on holds
// its own copy until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the
// device address is looked up once per device and used from then on.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes];
void* g_static_scratch_ptr[kMaxDevices] = {};
std::mutex g_static_scratch_mutex;

// Device address of the current device's copy of the scratch array, or null.
void* static_scratch() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_static_scratch_mutex);
    if (g_static_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch)) != hipSuccess) return nullptr;
        g_static_scratch_ptr[dev] = p;
    }
    return g_static_scratch_ptr[dev];
}

// Walks the workspace once; with base == nullptr it only measures.
struct Carver {
    char* base;
    size_t used = 0;
    explicit Carver(void* b) : base((char*)b) {}
    template <typename T>
    T* take(size_t count) {
        used = align_up(used, 256);
        T* p = base ? (T*)(base + used) : nullptr;
        used += count * sizeof(T);
        return p;
    }
};

struct Workspace {
    int32_t *topk_idx, *local_rank, *blk_hist, *hist_sums, *counts, *offsets, *perm, *inv_perm, *row_token, *sched;
    float *gates, *partial, *y_slot, *y_shared;
    void *act, *act_shared, *u;
    int slot_planes = 1, shared_planes = 1;   // planes of y_slot / y_shared the last launches wrote
    bool direct = false;                      // the routed down GEMM wrote the layer's output itself
    bool fused = false;                       // the caller launches down + combine as one kernel (run_experts stopped after gate/up)
    size_t bytes;
};

Workspace carve(const lexi_layer_t& ly, int T, int k, void* base) {
    Workspace w{};
    Carver c(base);
    const size_t A = (size_t)T * k;
    const size_t es = ly.dtype == LEXI_BF16 ? 2 : 4;
    // chained stack: the normalised MoE input.  First, so that its place does not depend on the layer or on k: a
    // block's combine writes the next block's input there.
    w.u = c.take<char>((size_t)T * ly.d * es);
    const size_t partial_at = align_up(c.used, 256);
    w.partial = c.take<float>((size_t)(ly.d / 128) * T * 64);
    w.local_rank = c.take<int32_t>(A);
    w.blk_hist = c.take<int32_t>(((size_t)T + 7) / 8 * 64);
    // What is written when the partials have been read shares their place: the expert table and, for many tokens, the sums of
    // the histograms.  Where router and top-k are one launch the partials stay in LDS, and the histograms (blocks of 4 tokens:
    // twice as many) take their place, with the table behind them.  Up to kFusedTailMaxT tokens there are neither ranks nor
    // histograms, and the table may run into their place.
    size_t sched_at = 0;
    if (T > kSmallRouterMaxT && T <= kFineRouterMaxT) {
        w.blk_hist = (int32_t*)w.partial;
        sched_at = ((size_t)T + 3) / 4 * 64;
    } else if (T <= kFusedTailMaxT) {
        const size_t room = (align_up(c.used, 256) - partial_at) / sizeof(int32_t);
        if (room < kSchedInts) c.take<int32_t>(kSchedInts - room);
    }
    w.topk_idx = c.take<int32_t>(A);
    w.gates = c.take<float>(A);
    w.counts = c.take<int32_t>(64);
    w.offsets = c.take<int32_t>(68);
    w.perm = c.take<int32_t>(A);
    w.inv_perm = c.take<int32_t>(A);
    w.row_token = c.take<int32_t>(A);
    if (base != nullptr) {
        w.sched = (int32_t*)w.partial + sched_at;
        w.hist_sums = w.sched + kSchedInts;   // (more than kPermuteDirectBlocks router blocks only: the partials are far longer)
    }
    w.act = c.take<char>(A * ly.F * es);
    // two planes wherever the down GEMM may split its reduction (independent of T and k, so that the size asked for
    // at (T_max, k_max) covers every smaller call)
    const bool bf = ly.dtype == LEXI_BF16;
    w.y_slot = c.take<float>(A * ly.d * ((bf && ksplit_eligible(ly.F)) ? 2 : 1));
    if (ly.F_shared > 0) {
        w.act_shared = c.take<char>((size_t)T * ly.F_shared * es);
        w.y_shared = c.take<float>((size_t)T * ly.d * ((bf && ksplit_eligible(ly.F_shared)) ? 2 : 1));
    }
    w.bytes = align_up(c.used, 256);
    return w;
}

inline bool misaligned(const void* p) { return ((uintptr_t)p & 15u) != 0; }

lexi_status check_layer(const lexi_layer_t* ly) {
    if (ly == nullptr) return LEXI_ERR_NULL;
    if (ly->dtype != LEXI_F32 && ly->dtype != LEXI_BF16) return LEXI_ERR_DTYPE;
    if (ly->shared_kind < LEXI_SHARED_NONE || ly->shared_kind > LEXI_SHARED_SIGMOID) return LEXI_ERR_DTYPE;
    if (ly->E < 1 || ly->E > 64) return LEXI_ERR_SHAPE;
    if (ly->d < 128 || ly->d % 128 != 0) return LEXI_ERR_SHAPE;
    if (ly->F < 64 || ly->F % 64 != 0) return LEXI_ERR_SHAPE;
    if (ly->F_shared < 0 || ly->F_shared % 64 != 0) return LEXI_ERR_SHAPE;
    if ((ly->F_shared > 0) != (ly->shared_kind != LEXI_SHARED_NONE)) return LEXI_ERR_SHAPE;
    if (!ly->w_router || !ly->w_gate || !ly->w_up || !ly->w_down) return LEXI_ERR_NULL;
    if (ly->F_shared > 0 && (!ly->ws_gate || !ly->ws_up || !ly->ws_down)) return LEXI_ERR_NULL;
    if (ly->shared_kind == LEXI_SHARED_SIGMOID && !ly->w_shared_gate) return LEXI_ERR_NULL;
    const void* ptrs[] = {ly->w_router, ly->router_bias, ly->w_gate, ly->w_up, ly->w_down,
                          ly->ws_gate, ly->ws_up, ly->ws_down, ly->w_shared_gate};
    for (const void* p : ptrs)
        if (p && misaligned(p)) return LEXI_ERR_ALIGN;
    return LEXI_OK;
}

// Limits on (T, k) that every entry point running the routed path shares.
lexi_status check_sizes(const lexi_layer_t* ly, int32_t T, int32_t k) {
    if (T < 0) return LEXI_ERR_SHAPE;
    if (k < 1 || k > ly->E) return LEXI_ERR_BAD_K;
    if ((int64_t)T * k >= (1 << 24)) return LEXI_ERR_SHAPE;
    // the bf16 GEMMs, on tiles and streaming, address their input rows with 32-bit byte offsets
    const uint64_t es = ly->dtype == LEXI_BF16 ? 2 : 4, lim = (uint64_t)1 << 32;
    if ((uint64_t)T * ly->d * es >= lim || (uint64_t)T * k * ly->F * es >= lim || (uint64_t)T * ly->F_shared * es >= lim)
        return LEXI_ERR_SHAPE;
    return LEXI_OK;
}

lexi_status check_call(const lexi_layer_t* ly, const void* x, const void* y, int32_t y_dtype, int32_t T, int32_t k,
                       const void* workspace, size_t workspace_bytes, const lexi_routing_out_t* dbg) {
    lexi_status st = check_layer(ly);
    if (st != LEXI_OK) return st;
    if (y_dtype != LEXI_F32 && y_dtype != LEXI_BF16) return LEXI_ERR_DTYPE;
    st = check_sizes(ly, T, k);
    if (st != LEXI_OK) return st;
    if (T == 0) return LEXI_OK;
    if (!x || !y || !workspace) return LEXI_ERR_NULL;
    if (misaligned(x) || misaligned(y) || misaligned(workspace)) return LEXI_ERR_ALIGN;
    if (dbg) {
        const void* ptrs[] = {dbg->topk_idx, dbg->gates, dbg->counts, dbg->offsets, dbg->perm, dbg->inv_perm, dbg->moe_input};
        for (const void* p : ptrs)
            if (p && misaligned(p)) return LEXI_ERR_ALIGN;
    }
    if (workspace_bytes < carve(*ly, T, k, nullptr).bytes) return LEXI_ERR_WORKSPACE;
    return LEXI_OK;
}

// Launch plan of the GEMMs of one call (what lexi_moe_gemm_plan and, its down part, lexi_moe_down_plan report).
struct LayerPlan {
    bool gateup_streams;                   // weight-streaming schedule instead of the tile schedule
    bool routed_streams, shared_streams;   // same, for the down GEMMs
    TilePlan gateup, shared_gateup;        // gate/up GEMMs on the tile schedule
    TilePlan routed, shared;               // down GEMMs on the tile schedule
    bool routed_direct;                    // with k == 1 and nothing to add: rows stored straight into y
    bool routed_fused;                     // a handful of tokens: down projections and combine in one launch
    bool f32_fused;                        // a small fp32 call: the same
};
LayerPlan plan_layer(const lexi_layer_t& ly, int32_t T, int32_t k, bool allow_split, bool allow_direct) {
    LayerPlan p{};
    const bool bf = ly.dtype == LEXI_BF16;
    const int64_t A = (int64_t)T * k;
    const int64_t few_items = (A / 128 + (A < ly.E ? A : ly.E)) * ((ly.d + 255) / 256);
    p.gateup_streams = !bf || A <= (int64_t)kStreamRowsPerExpert * ly.E;
    const bool direct = allow_direct && k == 1 && ly.F_shared == 0;
    p.routed_streams = p.gateup_streams || (few_items <= kStreamDownMaxItems && down_streams(A, ly.E, ly.F, ly.d, direct));
    p.shared_streams = !bf || T <= kStreamDenseRows;
    p.gateup = p.routed = p.shared = TilePlan{false, bf ? kTileRows : kF32TileRows, 1};
    p.shared_gateup = TilePlan{false, !bf ? kF32TileRows : T <= kSharedJoinsMaxT ? kSharedTileRows : kTileRows, 1};
    if (!p.gateup_streams) p.gateup = plan_gateup_tiles(A, ly.E, ly.d, ly.F);
    // (allow_direct: the caller wants nothing but y -- no slot rows, no residual, no normalised copy)
    p.routed_fused = bf && allow_direct && T <= kFusedDownMaxT && A <= kFusedDownMaxRows &&
                     (p.gateup_streams || few_items <= kStreamDownMaxItems) && ly.shared_kind != LEXI_SHARED_SIGMOID;
    if (p.routed_fused) p.routed_streams = true;
    p.f32_fused = !bf && allow_direct && ly.shared_kind != LEXI_SHARED_SIGMOID && f32_down_combine_fits(T, k, ly.d, ly.F, ly.F_shared);
    if (!p.routed_streams) {
        p.routed = plan_down_tiles(A, ly.E, ly.F, ly.d, allow_split, direct);
        p.routed_direct = direct && p.routed.ksplit == 1;
    }
    if (ly.F_shared > 0 && !p.shared_streams) {
        p.shared = plan_down_tiles(T, 1, ly.F_shared, ly.d, true, false);
        if (T <= kSharedJoinsMaxT) {
            const int rows = p.routed_streams ? kHalfTileRows : p.routed.wide ? kSharedTileRows : p.routed.tile_rows;
            p.shared = TilePlan{p.routed.wide, rows, p.shared.ksplit};
            if (!p.gateup_streams) p.shared_gateup.tile_rows = p.gateup.tile_rows;
        }
    }
    return p;
}

// Routing and the expert GEMMs of one layer at top-k = k: fills the routing arrays, act and y_slot of `w`, and (`with_shared`)
// act_shared and y_shared.
// `allow_split`: the down GEMM may write two planes of y_slot (w.slot_planes tells).  `direct_y` != null (k == 1, nothing
// else to add): the down GEMM stores the output rows straight into the layer's output (w.direct tells whether it did).
lexi_status run_experts(const lexi_layer_t& ly, const void* x, int32_t T, int32_t k, Workspace& w, hipStream_t s,
                        const lexi_stage_events_t* events, bool with_shared, bool allow_split = true, void* direct_y = nullptr,
                        bool direct_bf16 = false, bool chained = false) {
    auto mark = [&](int i) {
        if (events && events->ev[i]) (void)hipEventRecord((hipEvent_t)events->ev[i], s);
    };
    const bool bf = ly.dtype == LEXI_BF16;
    RoutingArgs r{};
    r.x = x; r.is_bf16 = bf; r.w_router = ly.w_router; r.bias = ly.router_bias;
    r.T = T; r.d = ly.d; r.E = ly.E; r.k = k;
    r.partial = w.partial; r.topk_idx = w.topk_idx; r.gates = w.gates; r.local_rank = w.local_rank; r.blk_hist = w.blk_hist;
    r.hist_sums = w.hist_sums;
    r.counts = w.counts; r.offsets = w.offsets; r.perm = w.perm; r.inv_perm = w.inv_perm; r.row_token = w.row_token;
    r.sched = w.sched;
    const int64_t A = (int64_t)T * k;
    const LayerPlan plan = plan_layer(ly, T, k, allow_split, direct_y != nullptr);
    r.plan.tile_rows[0] = plan.gateup.tile_rows;
    r.plan.tile_rows[1] = plan.routed.tile_rows;
    // up to 16 tokens on the streaming schedule: what follows the router's partials is part of the gate/up launch
    const bool select = bf && plan.gateup_streams && T <= kSelectMaxT;
    if ((select ? launch_router_partials(r, s) : launch_routing(r, s)) != hipSuccess) return LEXI_ERR_LAUNCH;
    mark(1);

    auto dense = [&](FfnArgs& f, int tile_rows) {   // the shared expert: one group of T rows
        f.is_bf16 = bf; f.M = T; f.chained = chained; f.tile_rows = tile_rows; f.max_tiles = (T + tile_rows - 1) / tile_rows;
    };
    FfnArgs g{}, sg{};
    g.streaming = plan.gateup_streams;
    g.chained = chained;
    g.is_bf16 = bf; g.in = x; g.row_token = w.row_token; g.in_rows = T; g.w0 = ly.w_gate; g.w1 = ly.w_up; g.K = ly.d;
    g.features = ly.F; g.M = (int)A; g.tile_rows = r.plan.tile_rows[0];
    g.max_tiles = (int)max_tiles(A, ly.E, g.tile_rows); g.sched = w.sched; g.out = w.act;
    dense(sg, plan.shared_gateup.tile_rows);
    sg.streaming = plan.shared_streams;
    sg.in = x; sg.w0 = ly.ws_gate; sg.w1 = ly.ws_up; sg.K = ly.d; sg.features = ly.F_shared; sg.out = w.act_shared;
    if ((select ? launch_select_gateup(r, g, with_shared ? &sg : nullptr, s) : launch_gateup(g, with_shared ? &sg : nullptr, s)) != hipSuccess)
        return LEXI_ERR_LAUNCH;
    mark(2);

    FfnArgs dn{}, sd{};
    dn.is_bf16 = bf; dn.in = w.act; dn.row_token = nullptr; dn.w0 = ly.w_down; dn.w1 = nullptr; dn.K = ly.F;
    dn.features = ly.d; dn.M = (int)A; dn.tile_rows = r.plan.tile_rows[1];
    dn.max_tiles = (int)max_tiles(A, ly.E, dn.tile_rows); dn.sched = w.sched; dn.out = w.y_slot;
    if (select) {   // (the work list would lie where other workgroups of that launch still read the partials)
        dn.sched = w.sched = nullptr;
        dn.counts = w.counts; dn.E = ly.E;
    }
    dn.streaming = plan.routed_streams;
    dn.chained = chained;
    dn.wide = plan.routed.wide;
    dn.ksplit = w.slot_planes = plan.routed.ksplit;
    dn.plane_stride = (size_t)A * ly.d;
    dense(sd, plan.shared.tile_rows);
    sd.streaming = plan.shared_streams;
    sd.in = w.act_shared; sd.w0 = ly.ws_down; sd.K = ly.F_shared; sd.features = ly.d; sd.out = w.y_shared;
    sd.wide = plan.shared.wide;
    sd.ksplit = w.shared_planes = plan.shared.ksplit;
    sd.plane_stride = (size_t)T * ly.d;
    w.direct = plan.routed_direct;
    w.fused = plan.routed_fused || plan.f32_fused;
    if (w.fused) return LEXI_OK;   // run_layer launches down (routed and shared) + combine
    if (plan.routed_direct) {
        dn.out = direct_y; dn.scatter = w.row_token; dn.out_bf16 = direct_bf16;
    }
    if (launch_down(dn, with_shared ? &sd : nullptr, s) != hipSuccess) return LEXI_ERR_LAUNCH;
    mark(3);
    return LEXI_OK;
}

// One layer, arguments already validated.
// `hidden` != null selects the chained block: the MoE input is `u_in` (the normalised hidden state, written by the
// caller or by the previous block's combine), the block's output is added to `hidden` (y may be `hidden` itself), and
// with `u_out` the combine also writes the next block's normalised input.
lexi_status run_layer(const lexi_layer_t& ly, const void* x, void* y, int32_t y_dtype, int32_t T, int32_t k,
                      void* workspace, hipStream_t s, const lexi_routing_out_t* dbg,
                      const lexi_stage_events_t* events = nullptr, const float* hidden = nullptr,
                      const void* u_in = nullptr, void* u_out = nullptr) {
    auto mark = [&](int i) {
        if (events && events->ev[i]) (void)hipEventRecord((hipEvent_t)events->ev[i], s);
    };
    mark(0);
    Workspace w = carve(ly, T, k, workspace);
    const bool bf = ly.dtype == LEXI_BF16;
    if (hidden != nullptr) {
        x = u_in;
    } else if (dbg && dbg->moe_input) {
        if (hipMemcpyAsync(dbg->moe_input, x, (size_t)T * ly.d * (bf ? 2 : 4), hipMemcpyDeviceToDevice, s) != hipSuccess)
            return LEXI_ERR_LAUNCH;
    }
    // routing results land directly in the caller's arrays when those are given
    if (dbg) {
        if (dbg->topk_idx) w.topk_idx = dbg->topk_idx;
        if (dbg->gates) w.gates = dbg->gates;
        if (dbg->counts) w.counts = dbg->counts;
        if (dbg->offsets) w.offsets = dbg->offsets;
        if (dbg->perm) w.perm = dbg->perm;
        if (dbg->inv_perm) w.inv_perm = dbg->inv_perm;
    }

    // Nothing but y to produce (no residual, no normalised copy): the routed down launch may write y itself -- with
    // one active expert and no shared one on the tile schedule, or for a handful of tokens with the combine fused in
    // (plan_layer decides).
    const bool direct = hidden == nullptr && u_out == nullptr;
    {
        const lexi_status st = run_experts(ly, x, T, k, w, s, events, ly.F_shared > 0, true, direct ? y : nullptr,
                                          y_dtype == LEXI_BF16, hidden != nullptr);
        if (st != LEXI_OK) return st;
    }
    if (w.fused) {
        // (one launch for both down projections and the combine: 3, 4 and 5 are recorded behind it)
        DownCombineArgs f{};
        f.act = w.act; f.w_down = ly.w_down; f.F = ly.F; f.d = ly.d; f.T = T; f.k = k; f.sched = w.sched;
        f.counts = w.counts; f.E = ly.E;
        f.inv_perm = w.inv_perm; f.gates = w.gates;
        if (ly.F_shared > 0) { f.act_shared = w.act_shared; f.ws_down = ly.ws_down; f.F_shared = ly.F_shared; }
        f.y = y; f.y_bf16 = y_dtype == LEXI_BF16;
        f.topk_idx = w.topk_idx;
        if ((bf ? launch_down_combine(f, s) : launch_down_combine_f32(f, s)) != hipSuccess) return LEXI_ERR_LAUNCH;
        for (int i : {3, 4, 5}) mark(i);
        return LEXI_OK;
    }

    mark(4);
    if (w.direct) {   // y is complete
        mark(5);
        return LEXI_OK;
    }

    CombineArgs c{};
    c.y_slot = w.y_slot; c.inv_perm = w.inv_perm; c.gates = w.gates;
    c.slot_planes = w.slot_planes; c.slot_plane_stride = (size_t)T * k * ly.d;
    c.shared_planes = w.shared_planes; c.shared_plane_stride = (size_t)T * ly.d;
    c.y_shared = ly.F_shared > 0 ? w.y_shared : nullptr;
    c.x = x; c.x_bf16 = bf;
    c.w_shared_gate = ly.shared_kind == LEXI_SHARED_SIGMOID ? ly.w_shared_gate : nullptr;
    c.residual = hidden; c.u_next = u_out;
    c.T = T; c.d = ly.d; c.k = k; c.y = y; c.y_bf16 = y_dtype == LEXI_BF16;
    if (launch_combine(c, s) != hipSuccess) return LEXI_ERR_LAUNCH;
    mark(5);
    return LEXI_OK;
}

}  // namespace

extern "C" {

lexi_status lexi_pack_weights(const void* src, void* dst, int64_t n_matrices, int32_t rows, int32_t K, int32_t dtype,
                              void* hip_stream) {
    if (dtype != LEXI_F32 && dtype != LEXI_BF16) return LEXI_ERR_DTYPE;
    if (n_matrices < 0 || rows < 16 || rows % 16 != 0 || K < 32 || K % 32 != 0) return LEXI_ERR_SHAPE;
    if (n_matrices == 0) return LEXI_OK;
    if (!src || !dst) return LEXI_ERR_NULL;
    if (misaligned(src) || misaligned(dst) || (dtype == LEXI_F32 && (((uintptr_t)src | (uintptr_t)dst) & 31u)))
        return LEXI_ERR_ALIGN;
    const size_t bytes = (size_t)n_matrices * rows * K * (dtype == LEXI_BF16 ? 2 : 4);
    const char *a = (const char*)src, *b = (const char*)dst;
    if (a < b + bytes && b < a + bytes) return LEXI_ERR_SHAPE;  // overlapping buffers
    if (launch_pack(src, dst, n_matrices, rows, K, dtype == LEXI_BF16, (hipStream_t)hip_stream) != hipSuccess)
        return LEXI_ERR_LAUNCH;
    return LEXI_OK;
}

size_t lexi_moe_workspace_bytes(const lexi_layer_t* layers, int32_t L, int32_t T_max, int32_t k_max) {
    if (!layers || L < 1 || T_max < 0 || k_max < 1) return 0;
    size_t need = 256;
    for (int l = 0; l < L; ++l) {
        if (check_layer(&layers[l]) != LEXI_OK) return 0;
        // a layer cannot be asked for more active experts than it has
        const size_t b = carve(layers[l], T_max, k_max < layers[l].E ? k_max : layers[l].E, nullptr).bytes;
        need = b > need ? b : need;
    }
    return need;
}

lexi_status lexi_moe_layer_forward(const lexi_layer_t* layer, const void* x, void* y, int32_t y_dtype, int32_t T,
                                   int32_t k, void* workspace, size_t workspace_bytes, void* hip_stream,
                                   const lexi_routing_out_t* dbg) {
    lexi_status st = check_call(layer, x, y, y_dtype, T, k, workspace, workspace_bytes, dbg);
    if (st != LEXI_OK || T == 0) return st;
    return run_layer(*layer, x, y, y_dtype, T, k, workspace, (hipStream_t)hip_stream, dbg);
}

lexi_status lexi_moe_layer_forward_static(const lexi_layer_t* layer, const void* x, void* y, int32_t y_dtype, int32_t T,
                                          int32_t k, void* hip_stream, const lexi_routing_out_t* dbg) {
    // validate against the static array's size first: a fake non-null, aligned workspace address stands in until the
    // real one is looked up (check_call only compares it with null and tests its alignment)
    lexi_status st = check_call(layer, x, y, y_dtype, T, k, (const void*)(uintptr_t)256, kStaticScratchBytes, dbg);
    if (st != LEXI_OK || T == 0) return st;
    void* ws = static_scratch();
    if (ws == nullptr) return LEXI_ERR_LAUNCH;
    // every kernel writes the part of the scratch it reads later in the same call, so nothing needs clearing
    return run_layer(*layer, x, y, y_dtype, T, k, ws, (hipStream_t)hip_stream, dbg);
}

lexi_status lexi_moe_stack_forward_profiled(const lexi_layer_t* layers, int32_t L, const int32_t* k_vec,
                                            const void* x, int64_t x_layer_stride, void* y, int64_t y_layer_stride,
                                            int32_t y_dtype, int32_t T, int32_t mode, void* workspace,
                                            size_t workspace_bytes, void* hip_stream,
                                            const lexi_routing_out_t* dbg_per_layer,
                                            const lexi_stage_events_t* events_per_layer) {
    if (!layers || !k_vec) return LEXI_ERR_NULL;
    if (L < 1 || x_layer_stride < 0 || y_layer_stride < 0) return LEXI_ERR_SHAPE;
    if (mode != LEXI_STACK_INDEPENDENT && mode != LEXI_STACK_CHAINED) return LEXI_ERR_DTYPE;
    const bool chained = mode == LEXI_STACK_CHAINED;
    if (chained && (y_dtype != LEXI_F32 || x_layer_stride != 0)) return LEXI_ERR_DTYPE;   // fp32 hidden state, one input
    // validate every layer before the first launch: an error must leave nothing enqueued
    for (int l = 0; l < L; ++l) {
        const size_t xes = layers[l].dtype == LEXI_BF16 ? 2 : 4;
        const size_t yes = y_dtype == LEXI_BF16 ? 2 : 4;
        const void* xl = x ? (const char*)x + (size_t)l * x_layer_stride * xes : nullptr;
        const void* yl = y ? (const char*)y + (size_t)l * y_layer_stride * yes : nullptr;
        lexi_status st = check_call(&layers[l], xl, yl, y_dtype, T, k_vec[l], workspace, workspace_bytes,
                                    dbg_per_layer ? &dbg_per_layer[l] : nullptr);
        if (st != LEXI_OK) return st;
        if (chained) {
            // one hidden state flows through all blocks: same width and dtype everywhere; outputs either all in one
            // buffer (stride 0: only the last survives) or one full buffer per layer
            if (layers[l].d != layers[0].d || layers[l].dtype != layers[0].dtype) return LEXI_ERR_SHAPE;
            if (y_layer_stride != 0 && y_layer_stride < (int64_t)T * layers[l].d) return LEXI_ERR_SHAPE;
        } else if (L > 1 && T > 0 && y_layer_stride < (int64_t)T * layers[l].d) {
            return LEXI_ERR_SHAPE;  // outputs would overlap
        }
    }
    if (T == 0) return LEXI_OK;
    hipStream_t s = (hipStream_t)hip_stream;
    if (chained) {
        // h_0 = x, widened into the first output buffer; block l reads h_l where block l-1 left it and writes h_{l+1}.
        // The normalised input of block 0 comes from its own kernel, that of every later block from the combine of
        // the block before it; it lives at the start of the workspace unless the caller asked to see it.
        const bool bf = layers[0].dtype == LEXI_BF16;
        auto u_of = [&](int l) -> void* {
            return (dbg_per_layer && dbg_per_layer[l].moe_input) ? dbg_per_layer[l].moe_input : workspace;
        };
        float* h = (float*)y;
        if (launch_start_chain(x, bf, T, layers[0].d, kRmsEps, h, u_of(0), s) != hipSuccess) return LEXI_ERR_LAUNCH;
        for (int l = 0; l < L; ++l) {
            float* h_out = (float*)y + (size_t)l * y_layer_stride;
            lexi_status st = run_layer(layers[l], nullptr, h_out, LEXI_F32, T, k_vec[l], workspace, s,
                                       dbg_per_layer ? &dbg_per_layer[l] : nullptr,
                                       events_per_layer ? &events_per_layer[l] : nullptr, h, u_of(l),
                                       l + 1 < L ? u_of(l + 1) : nullptr);
            if (st != LEXI_OK) return st;
            h = h_out;
        }
        return LEXI_OK;
    }
    for (int l = 0; l < L; ++l) {
        const size_t xes = layers[l].dtype == LEXI_BF16 ? 2 : 4;
        const size_t yes = y_dtype == LEXI_BF16 ? 2 : 4;
        const void* xl = (const char*)x + (size_t)l * x_layer_stride * xes;
        void* yl = (char*)y + (size_t)l * y_layer_stride * yes;
        lexi_status st = run_layer(layers[l], xl, yl, y_dtype, T, k_vec[l], workspace, s,
                                   dbg_per_layer ? &dbg_per_layer[l] : nullptr,
                                   events_per_layer ? &events_per_layer[l] : nullptr);
        if (st != LEXI_OK) return st;
    }
    return LEXI_OK;
}

lexi_status lexi_moe_stack_forward(const lexi_layer_t* layers, int32_t L, const int32_t* k_vec, const void* x,
                                   int64_t x_layer_stride, void* y, int64_t y_layer_stride, int32_t y_dtype,
                                   int32_t T, int32_t mode, void* workspace, size_t workspace_bytes,
                                   void* hip_stream, const lexi_routing_out_t* dbg_per_layer) {
    return lexi_moe_stack_forward_profiled(layers, L, k_vec, x, x_layer_stride, y, y_layer_stride, y_dtype, T, mode,
                                           workspace, workspace_bytes, hip_stream, dbg_per_layer, nullptr);
}

size_t lexi_moe_profile_workspace_bytes(const lexi_layer_t* layer, int32_t T_max, int32_t k_base, int32_t n_k) {
    if (!layer || check_layer(layer) != LEXI_OK || T_max < 0 || k_base < 1 || k_base > layer->E || n_k < 1 ||
        n_k > kProfileMaxK)
        return 0;
    return carve(*layer, T_max, k_base, nullptr).bytes + align_up((size_t)n_k * T_max * sizeof(float), 256);
}

lexi_status lexi_moe_profile_layer(const lexi_layer_t* layer, const void* x, int32_t T, int32_t k_base,
                                   const int32_t* k_list, int32_t n_k, float* delta, void* workspace,
                                   size_t workspace_bytes, void* hip_stream) {
    lexi_status st = check_layer(layer);
    if (st != LEXI_OK) return st;
    if (!k_list || !delta) return LEXI_ERR_NULL;
    if (T < 1 || n_k < 1 || n_k > kProfileMaxK) return LEXI_ERR_SHAPE;
    st = check_sizes(layer, T, k_base);
    if (st != LEXI_OK) return st;
    ProfileKList kl{};
    kl.n = n_k;
    for (int i = 0; i < n_k; ++i) {
        if (k_list[i] < 1 || k_list[i] > k_base) return LEXI_ERR_BAD_K;
        kl.k[i] = k_list[i];
    }
    if (!x || !workspace) return LEXI_ERR_NULL;
    if (misaligned(x) || misaligned(workspace) || misaligned(delta)) return LEXI_ERR_ALIGN;
    Workspace w = carve(*layer, T, k_base, workspace);
    if (workspace_bytes < w.bytes + align_up((size_t)n_k * T * sizeof(float), 256)) return LEXI_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    st = run_experts(*layer, x, T, k_base, w, s, nullptr, /*with_shared=*/false, /*allow_split=*/false);
    if (st != LEXI_OK) return st;
    ProfileArgs p{};
    p.y_slot = w.y_slot; p.inv_perm = w.inv_perm; p.gates = w.gates;
    p.T = T; p.d = layer->d; p.k_base = k_base; p.klist = kl;
    p.part = (float*)((char*)workspace + w.bytes);
    p.delta = delta;
    return launch_profile(p, s) == hipSuccess ? LEXI_OK : LEXI_ERR_LAUNCH;
}

int32_t lexi_moe_down_plan(const lexi_layer_t* layer, int32_t T, int32_t k, int32_t which) {
    if (check_layer(layer) != LEXI_OK || T < 1 || k < 1 || k > layer->E) return -1;
    const LayerPlan p = plan_layer(*layer, T, k, true, true);
    if (layer->dtype != LEXI_BF16) {
        // the sizes at which bf16 layers once changed schedule; whether the combine is in the same launch (f32_fused) is not told here
        const int64_t A = (int64_t)T * k, E = layer->E;
        if (which == 1) return layer->F_shared == 0 ? -1 : (T <= kStreamDenseRows ? 0 : 1);
        return which != 0 ? -1 : (A <= kStreamRowsPerExpert * E || max_tiles(A, layer->E, 128) * ((layer->d + 255) / 256) <= kStreamDownMaxItems) ? 0 : 1;
    }
    switch (which) {
        case 0: return p.routed_fused ? 4 : (p.routed_streams ? 0 : (p.routed_direct ? 3 : p.routed.ksplit));
        case 1: return layer->F_shared == 0 ? -1 : (p.shared_streams ? 0 : p.shared.ksplit);
        default: return -1;
    }
}

lexi_status lexi_moe_gemm_plan(const lexi_layer_t* layer, int32_t T, int32_t k, int32_t chained, int32_t which,
                               lexi_gemm_plan_t* out) {
    if (out == nullptr) return LEXI_ERR_NULL;
    lexi_status st = check_layer(layer);
    if (st == LEXI_OK) st = check_sizes(layer, T, k);
    if (st != LEXI_OK) return st;
    if (T < 1 || which < 0 || which > 3 || (which >= 2 && layer->F_shared == 0)) return LEXI_ERR_SHAPE;
    const LayerPlan p = plan_layer(*layer, T, k, true, !chained);
    const bool shared = which >= 2, down = which & 1;
    const TilePlan& t = shared ? (down ? p.shared : p.shared_gateup) : (down ? p.routed : p.gateup);
    *out = lexi_gemm_plan_t{};
    out->streams = shared ? p.shared_streams : down ? p.routed_streams : p.gateup_streams;
    out->tile_rows = t.tile_rows;
    out->ksplit = t.ksplit;
    out->direct = down && !shared && p.routed_direct;
    out->fused = down && !shared && (p.routed_fused || p.f32_fused);
    if (down && p.routed_fused) {
        out->waves = down_combine_features(layer->d);
    } else if (down && p.f32_fused) {
        const int slots = k + (layer->F_shared > 0 ? 1 : 0);
        out->waves = slots < 16 ? slots : 16;
    } else if (!out->streams) {
        out->waves = t.wide ? 8 : 4;
    } else {
        // the two jobs as the launcher sees them; a streaming one has four waves beside a tiled one in the same launch
        const bool bf = layer->dtype == LEXI_BF16;
        FfnArgs r{}, sh{};
        auto fill = [&](FfnArgs& f, const TilePlan& tp, bool streaming, int F, int64_t tiles) {
            f.is_bf16 = bf; f.streaming = streaming; f.wide = tp.wide; f.chained = chained != 0;
            f.K = down ? F : layer->d; f.features = down ? layer->d : F; f.max_tiles = (int)tiles;
        };
        const TilePlan &tr = down ? p.routed : p.gateup, &ts = down ? p.shared : p.shared_gateup;
        fill(r, tr, down ? p.routed_streams : p.gateup_streams, layer->F, max_tiles((int64_t)T * k, layer->E, tr.tile_rows));
        fill(sh, ts, p.shared_streams, layer->F_shared, (T + ts.tile_rows - 1) / ts.tile_rows);
        const bool joined = layer->F_shared > 0 && ffn_joins(r, sh);
        if (!bf || (joined && !(r.streaming && sh.streaming))) out->waves = 4;
        else out->waves = joined ? stream_launch_waves(r, &sh) : streamed_parts(shared ? sh : r);
    }
    return LEXI_OK;
}

const char* lexi_strerror(int32_t status) {
    switch (status) {
        case LEXI_OK: return "ok";
        case LEXI_ERR_NULL: return "a required pointer is NULL";
        case LEXI_ERR_SHAPE: return "a dimension violates the shape limits";
        case LEXI_ERR_BAD_K: return "k outside 1..E";
        case LEXI_ERR_DTYPE: return "unknown dtype, shared_kind or mode";
        case LEXI_ERR_WORKSPACE: return "workspace too small";
        case LEXI_ERR_ALIGN: return "a device pointer is not 16-byte aligned";
        case LEXI_ERR_LAUNCH: return "the HIP runtime refused a kernel launch";
        default: return "unknown status";
    }
}

const char* lexi_moe_version(void) { return "lexi-moe gfx950 0.1"; }

}  // extern "C"
