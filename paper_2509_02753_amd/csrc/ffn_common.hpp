// Pieces shared by the expert-FFN translation units: K-stage size, the packed weight layout, the tile schedule.
#pragma once
#include "kernels.hpp"

namespace lexi {

constexpr int BK = 64;         // K elements per LDS stage
constexpr int LDS_PAD = 8;     // bf16 elements of padding per LDS row (16 B): spreads the 16-byte operand reads over banks
constexpr int LDS_LD = BK + LDS_PAD;

// Expert weight matrices W[R][K] (R output features, K inputs) are stored in the MFMA-native "packed" layout:
// the matrix is cut into blocks of 16 rows x 32 K elements; a block is 64 runs of 8 consecutive K elements, run
// (q, i) = (K-octet q of the block, row i of the block) at position q*16 + i; blocks follow each other along K, then
// along R.  A wave-wide 16-byte-per-lane load of one block is therefore 1 KB of contiguous memory and is, as it
// stands, the A operand of v_mfma_f32_16x16x32_bf16 (lane = q*16 + i).
__host__ __device__ __forceinline__ size_t packed_index(int r, int k, int K) {
    return ((((size_t)(r >> 4) * (K >> 5) + (k >> 5)) * 64 + ((k & 31) >> 3) * 16 + (r & 15)) << 3) + (k & 7);
}

struct TileInfo {
    int expert, row0, rows;
};

// One grouped GEMM as the kernels see it (FfnArgs).  A launch takes two: the routed experts' and, in the blocks before it, the
// shared expert's.
struct FfnJob {
    const void* in;
    const int32_t* row_token;
    const void *w0, *w1;
    const int32_t *sched, *scatter, *counts;
    void* out;
    size_t plane_stride;
    int K, features, M, tile_rows, ksplit, out_bf16, E;
    int streams;              // taken by the weight-streaming schedule, blocks ordered (tile, unit of 16 features)
    int parts;                // there: parts a sum is taken in (streamed_parts)
    int blocks;               // workgroups of this job, a multiple of kXcds where a second job follows
};
inline FfnJob make_job(const FfnArgs& a, int blocks) {
    return FfnJob{a.in, a.row_token, a.w0, a.w1, a.sched, a.scatter, a.counts, a.out, a.plane_stride, a.K, a.features, a.M, a.tile_rows,
                  a.ksplit > 1 ? a.ksplit : 1, a.out_bf16 ? 1 : 0, a.E, a.streaming ? 1 : 0, streamed_parts(a), blocks};
}
// (by value: a conditional expression on two members would select between their addresses)
template <typename T>
__device__ __forceinline__ T choose(bool c, T a, T b) { return c ? a : b; }
// The job block `block` belongs to (wave-uniform); `block` is then counted from the job's first.
__device__ __forceinline__ FfnJob pick_job(const FfnJob& routed, const FfnJob& shared, int& block) {
    const bool first = block < shared.blocks;
    if (!first) block -= shared.blocks;
    FfnJob j;
    j.in = choose(first, shared.in, routed.in);
    j.row_token = choose(first, shared.row_token, routed.row_token);
    j.w0 = choose(first, shared.w0, routed.w0);
    j.w1 = choose(first, shared.w1, routed.w1);
    j.sched = choose(first, shared.sched, routed.sched);
    j.scatter = choose(first, shared.scatter, routed.scatter);
    j.counts = choose(first, shared.counts, routed.counts);
    j.E = choose(first, shared.E, routed.E);
    j.out = choose(first, shared.out, routed.out);
    j.plane_stride = choose(first, shared.plane_stride, routed.plane_stride);
    j.K = choose(first, shared.K, routed.K);
    j.features = choose(first, shared.features, routed.features);
    j.M = choose(first, shared.M, routed.M);
    j.tile_rows = choose(first, shared.tile_rows, routed.tile_rows);
    j.ksplit = choose(first, shared.ksplit, routed.ksplit);
    j.out_bf16 = choose(first, shared.out_bf16, routed.out_bf16);
    j.streams = choose(first, shared.streams, routed.streams);
    j.parts = choose(first, shared.parts, routed.parts);
    j.blocks = choose(first, shared.blocks, routed.blocks);
    return j;
}
inline int round_to_xcds(long long blocks) { return (int)((blocks + kXcds - 1) / kXcds * kXcds); }

// Tile t of the n = ceil(rows / tile height) tiles of a group: the group's 16-row blocks are dealt out evenly (heights
// differ by one block at most), so no tile is a short remainder that streams a whole weight slab for a few rows.
__device__ __forceinline__ void even_tile(int group_row0, int group_rows, int t, int n, TileInfo& ti) {
    const int nb = (group_rows + 15) >> 4;
    const int per = nb / n, extra = nb - per * n;
    const int b0 = t * per + min(t, extra);
    const int blocks = per + (t < extra ? 1 : 0);
    ti.row0 = group_row0 + b0 * 16;
    ti.rows = min(blocks * 16, group_rows - b0 * 16);
}

// The group token tile `tile` of GEMM G belongs to: its rows, its tiles [first, first + n).  One lane per expert looks, all
// lanes of the wave call it with the same tile.  sched == null: one dense group of M rows.
struct TileGroup {
    int expert, row0, rows, first, n;
};
template <int G>
__device__ __forceinline__ bool fetch_group(const int32_t* sched, int tile, int M, int tile_rows, TileGroup& g) {
    if (sched == nullptr) {
        g = TileGroup{0, 0, M, 0, (M + tile_rows - 1) / tile_rows};
        return tile < g.n;
    }
    if (tile >= sched[kSchedTiles + 64 * G + 63]) return false;        // (a scalar load: most workgroups of a small batch end here)
    const int lane = threadIdx.x & 63;
    const int off = sched[kSchedOff + lane], cnt = sched[kSchedCount + lane];
    const int end = sched[kSchedTiles + 64 * G + lane];     // tiles of experts 0 .. lane
    const int e = __builtin_amdgcn_readfirstlane(__popcll(__ballot(end <= tile)));
    g.expert = e;
    g.row0 = __builtin_amdgcn_readlane(off, e);
    g.rows = __builtin_amdgcn_readlane(cnt, e);
    g.first = e > 0 ? __builtin_amdgcn_readlane(end, e - 1) : 0;
    g.n = __builtin_amdgcn_readlane(end, e) - g.first;
    return true;
}

// The expert table of at most kSelectMaxT tokens from the experts' counts alone, lane = expert: rows, first row, and the number of
// experts with rows up to and with this one (each has one tile).
__device__ __forceinline__ void expert_table(const int32_t* counts, int E, int& count, int& offset, int& end) {
    const int lane = threadIdx.x & 63;
    count = lane < E ? counts[lane] : 0;
    offset = wave_inclusive_sum(count) - count;
    end = wave_inclusive_sum(count > 0 ? 1 : 0);
}

template <int G>
__device__ __forceinline__ bool fetch_tile(const FfnJob& j, int tile, TileInfo& ti) {
    TileGroup g;
    if (j.counts != nullptr) {
        int count, offset, end;
        expert_table(j.counts, j.E, count, offset, end);
        if (tile >= __builtin_amdgcn_readlane(end, 63)) return false;
        const int e = __builtin_amdgcn_readfirstlane(__popcll(__ballot(end <= tile)));
        ti = TileInfo{e, __builtin_amdgcn_readlane(offset, e), __builtin_amdgcn_readlane(count, e)};
        return true;
    }
    if (!fetch_group<G>(j.sched, tile, j.M, j.tile_rows, g)) return false;
    ti.expert = g.expert;
    ti.row0 = g.row0;
    ti.rows = g.rows;
    if (g.n > 1) even_tile(g.row0, g.rows, tile - g.first, g.n, ti);
    return true;
}

// XCD-aware work order for the tile kernels.  Workgroup ids are handed to the 8 XCDs round-robin (id % 8), each XCD
// with its own L2, and a CU holds two workgroups of four waves, so 64 consecutive work items of an XCD are resident
// together.  Work items are (token tile, column block).  They are ordered expert by expert; inside an expert by groups of
// kCbGroup column blocks; inside a group tile-major.  A window of 64 items then holds few distinct weight slabs,
// each read by ALL token tiles of its expert at the same time, whatever the number of column blocks is (sharing the
// weight stream is what pays: groups of 1 or 2 column blocks measured 10 to 40 % faster than groups of 8 or more,
// which favour sharing the much smaller token tile).  The item list is cut into 8 contiguous parts of equal length, XCD x
// takes the x-th.  (Parts of equal estimated cost measured up to 60 % slower: a part only slightly longer than the average
// needs a whole further round of its XCD's workgroup slots.)
// The grid is 1-D: 8 * ceil(ncb * max_tiles / 8) workgroups, times ksplit; `block` is the workgroup's number in its job.
constexpr int kCbGroup = 2;

// With ksplit > 1 every item appears ksplit times in a row, once per part of the reduction dimension.
template <int G>
__device__ __forceinline__ bool fetch_item(int block, const int32_t* sched, int ncb, int M, int tile_rows, int ksplit, TileInfo& ti,
                                           int& cb, int& part) {
    const int xcd = block % kXcds, slot = block / kXcds;
    const int ntiles = sched != nullptr ? sched[kSchedTiles + 64 * G + 63] : (M + tile_rows - 1) / tile_rows;
    const int total = ntiles * ncb * ksplit;
    const int per = (total + kXcds - 1) / kXcds;
    const int piece = xcd * per + slot;
    if (slot >= per || piece >= total) return false;
    const int item = piece / ksplit;
    part = piece - item * ksplit;
    // an expert with n tiles owns n * ncb consecutive items, so tile (item / ncb) belongs to the item's expert
    TileGroup g;
    if (!fetch_group<G>(sched, item / ncb, M, tile_rows, g)) return false;
    const int j = item - g.first * ncb;
    const int gsz = g.n * kCbGroup;
    const int q = j / gsz, r = j - q * gsz;
    const int gw = min(kCbGroup, ncb - q * kCbGroup);   // the last group of an expert may be narrower
    const int t = r / gw;
    cb = q * kCbGroup + (r - t * gw);
    ti.expert = g.expert;
    even_tile(g.row0, g.rows, t, g.n, ti);
    return true;
}

// Weight-streaming schedule: one unit of 16 output features of one token tile, by a workgroup of NW waves; red is LDS.
// `row_of(r)`: the row of `in` behind the tile's row r.  MAXB: 16-row blocks a tile holds at most.
template <int N> struct IntTag { static constexpr int value = N; };

// Four features of an output row: act = silu(g) * u in bf16, or g.
template <bool GATEUP>
__device__ __forceinline__ void store_unit(void* out, size_t at, const f32x4_t& g, const f32x4_t& u) {
    if (GATEUP) {
        u32x2_t pk;
        pk[0] = pack_bf16x2(silu(g[0]) * u[0], silu(g[1]) * u[1]);
        pk[1] = pack_bf16x2(silu(g[2]) * u[2], silu(g[3]) * u[3]);
        *(u32x2_t*)((bf16_t*)out + at) = pk;
    } else {
        *(f32x4_t*)((float*)out + at) = g;
    }
}

// K blocks [kb0, kb1) of a unit by one wave: NM weight matrices (w: their blocks 0 of the unit) against NTB row blocks (a lane's row of `in`
// at byte xoff), summed into acc in ascending order; `before(kb)` is called in front of a block's multiply-adds.
// Bound by round trips to memory, so the loads of U blocks are in flight all the time: a block's registers are loaded again, U blocks
// ahead, as soon as it has been multiplied.  (Places of the last round past the end load the last block again, unused: branch-free.)
// A part of fewer blocks loads only those it has: empty places took a tenth to a quarter of the launches of small layers (18 tokens, 12 experts, d
// 256, F 128: gate/up 5.2 -> 4.0 us; 21 tokens, 24 experts, d 512: gate/up 5.2 -> 4.4, down 4.4 -> 3.6; calls 2 to 8 %).
// The scheduling barriers keep the loads where they stand: left to itself the compiler saves registers and waits for nearly
// every block by itself (8 blocks in 7 to 10 round trips).  Launches before and after, us: down, 16 tokens, d 2048, K 1408, k 2 / 6 17.2 -> 14.6, 35.7 ->
// 30.2, 20 tokens, 64 experts 59.2 -> 48.7; gate/up, 1 token, k 6 21.2 -> 18.8, 20 tokens 97.8 -> 91.3, 30 tokens of d 1536 20.1 -> 16.0;
// beside tiles: down, 64 tokens, shared K 5632 74.6 -> 67.3, 100 tokens, k = 1 58.6 -> 51.7.
template <int NM, int NTB, int U, typename Before>
__device__ __forceinline__ void stream_blocks(const char* const (&w)[NM], const char* in, const uint32_t (&xoff)[NTB], int kb0, int kb1,
                                              f32x4_t (&acc)[NM][NTB], Before before) {
    // (known from here on only: the compiler would compute every place's addresses in front of the caller's loop over rows, in 20 registers)
    asm volatile("" : "+s"(kb0), "+s"(kb1));
    const uint32_t lane16 = (threadIdx.x & 63) * 16;
    bf16x8_t wr[U][NM], xr[U][NTB];
    auto load = [&](int u, int kb) {
        const char* x = in + (size_t)(uint32_t)kb * 64;
#pragma unroll
        for (int m = 0; m < NM; ++m) wr[u][m] = *(const bf16x8_t*)(w[m] + (size_t)(uint32_t)kb * 1024 + lane16);
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) xr[u][tb] = *(const bf16x8_t*)(x + xoff[tb]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int u, int kb) {
        before(kb);
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
            for (int m = 0; m < NM; ++m) acc[m][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[u][m], xr[u][tb], acc[m][tb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    if (kb1 - kb0 < U) {                 // (never with U = 1: the part has blocks)
#pragma unroll
        for (int u = 0; u < U - 1; ++u) {
            if (kb0 + u >= kb1) break;
            load(u, kb0 + u);
        }
#pragma unroll
        for (int u = 0; u < U - 1; ++u) {
            if (kb0 + u >= kb1) return;
            multiply(u, kb0 + u);
        }
        return;
    }
    int kb = kb0;
#pragma unroll
    for (int u = 0; u < U; ++u) load(u, kb + u);
    for (; kb + U < kb1; kb += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            multiply(u, kb + u);
            load(u, min(kb + U + u, kb1 - 1));
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (kb + u >= kb1) return;
        multiply(u, kb + u);
    }
}
// The same, as many blocks deep as REGS registers hold, 8 at most.  Eight row blocks leave one (its nine or ten loads fly together, none ahead),
// still less time than the plain loop (64 experts, k 1, 97 to 128 tokens, nearly all of one expert, d 1024 to 4096: whole calls 0.65 to 0.75
// times).  Where the depth would be 3 (down, four row blocks) or 5 (down, two; gate/up, one) a part of
// 4n or 4n - 1 blocks takes 4: a place of row blocks that is loaded for nothing costs more than the depth gives (down: 60 tokens, one
// expert, K 1408, parts of 5 and 6 blocks, the call 4 deep 211 us, 3 deep 200; 56 tokens, K 1920, parts of 7 and 8, the launch 10.7 and 11.4).
template <int NM, int NTB, int REGS, typename Before>
__device__ __forceinline__ void stream_part(const char* const (&w)[NM], const char* in, const uint32_t (&xoff)[NTB], int kb0, int kb1,
                                            f32x4_t (&acc)[NM][NTB], Before before) {
    constexpr int N = REGS / (4 * (NM + NTB)), U = N < 1 ? 1 : N > 8 ? 8 : N;
    if constexpr (U == 3 || U == 5) {
        if (((kb1 - kb0) & 3) == 0 || ((kb1 - kb0) & 3) == 3) {
            stream_blocks<NM, NTB, 4>(w, in, xoff, kb0, kb1, acc, before);
            return;
        }
    }
    stream_blocks<NM, NTB, U>(w, in, xoff, kb0, kb1, acc, before);
}

template <bool GATEUP, int NW, int MAXB, int REGS, typename RowOf>
__device__ __forceinline__ void stream_unit(const FfnJob& j, const TileInfo& tile, int unit, f32x4_t (*red)[2][64], RowOf row_of) {
    constexpr int NM = GATEUP ? 2 : 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int K = j.K, features = j.features, nkb = K >> 5;
    void* out = j.out;
    TileInfo ti = tile;
    const int kb0 = wave * nkb / NW, kb1 = (wave + 1) * nkb / NW;
    const size_t slab = ((size_t)(uint32_t)ti.expert * (features >> 4) + unit) * ((size_t)K * 32);
    const char* w[NM] = {(const char*)j.w0 + slab};
    if constexpr (GATEUP) w[1] = (const char*)j.w1 + slab;

    auto body = [&](auto ntb_tag) {
        constexpr int NTB = decltype(ntb_tag)::value;
        uint32_t xoff[NTB];
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
            const int rr = min(tb * 16 + l16, ti.rows - 1);  // rows past the group end re-read its last row; never stored
            xoff[tb] = (uint32_t)row_of(ti.row0 - tile.row0 + rr) * (uint32_t)(K * 2) + kq * 16;
        }
        f32x4_t acc[NM][NTB];
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) acc[m][tb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (kb0 < kb1) stream_part<NM, NTB, REGS>(w, (const char*)j.in, xoff, kb0, kb1, acc, [](int) {});
        // split-K reduction in wave order, one token block at a time; wave (tb % waves) finishes block tb
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
#pragma unroll
            for (int m = 0; m < NM; ++m) red[wave][m][lane] = acc[m][tb];
            __syncthreads();
            if (wave == tb % NW) {
                f32x4_t g = red[0][0][lane], u = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int v = 1; v < NW; ++v) g += red[v][0][lane];
                if (GATEUP) {
                    u = red[0][1][lane];
#pragma unroll
                    for (int v = 1; v < NW; ++v) u += red[v][1][lane];
                }
                // lane owns token (lane % 16), features 4*(lane/16) + 0..3 of the unit
                if (tb * 16 + l16 < ti.rows) store_unit<GATEUP>(out, (size_t)(ti.row0 + tb * 16 + l16) * features + unit * 16 + kq * 4, g, u);
            }
            __syncthreads();
        }
    };
    // 128 rows at a time (a tile may be taller; the second pass over the weights is then served by the cache)
    const int row_end = ti.row0 + ti.rows;
    for (; ti.row0 < row_end; ti.row0 += 128) {
        ti.rows = min(128, row_end - ti.row0);
        const int ntb = (ti.rows + 15) >> 4;
        if constexpr (MAXB == 1) {
            body(IntTag<1>{});
        } else {
            if (ntb <= 1) body(IntTag<1>{});
            else if (ntb <= 2) body(IntTag<2>{});
            else if (ntb <= 4) body(IntTag<4>{});
            else body(IntTag<8>{});
        }
    }
}

// The same with the sum in eight parts by a workgroup of four waves: a wave takes two parts, whose blocks follow each other, in one stream of
// loads.  All parts of up to MAXB row blocks meet in LDS at once (stream_eight_lds), and a wave finishes one block.
template <bool GATEUP> constexpr int stream_eight_lds(int maxb) { return 8 * maxb * (GATEUP ? 2 : 1) * 64; }   // f32x4_t's

template <bool GATEUP, int MAXB, int REGS, typename RowOf>
__device__ __forceinline__ void stream_unit_eight(const FfnJob& j, const TileInfo& tile, int unit, f32x4_t* red, RowOf row_of) {
    static_assert(MAXB <= 4, "a wave finishes one row block");
    constexpr int NM = GATEUP ? 2 : 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int K = j.K, features = j.features, nkb = K >> 5;
    TileInfo ti = tile;
    const size_t slab = ((size_t)(uint32_t)ti.expert * (features >> 4) + unit) * ((size_t)K * 32);
    const char* w[NM] = {(const char*)j.w0 + slab};
    if constexpr (GATEUP) w[1] = (const char*)j.w1 + slab;
    const int kb0 = 2 * wave * nkb / 8, second = (2 * wave + 1) * nkb / 8, kb1 = (2 * wave + 2) * nkb / 8;

    auto body = [&](auto ntb_tag) {
        constexpr int NTB = decltype(ntb_tag)::value;
        auto at = [&](int part, int tb, int m) { return red + (((part * NTB + tb) * NM + m) * 64 + lane); };
        uint32_t xoff[NTB];
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
            const int rr = min(tb * 16 + l16, ti.rows - 1);  // rows past the group end re-read its last row; never stored
            xoff[tb] = (uint32_t)row_of(ti.row0 - tile.row0 + rr) * (uint32_t)(K * 2) + kq * 16;
        }
        f32x4_t acc[NM][NTB];
        auto store_part = [&](int part) {                    // and start the next
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    *at(part, tb, m) = acc[m][tb];
                    acc[m][tb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
                }
        };
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) acc[m][tb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (second == kb0) store_part(2 * wave);             // (an empty first part)
        if (kb0 < kb1)
            stream_part<NM, NTB, REGS>(w, (const char*)j.in, xoff, kb0, kb1, acc, [&](int kb) {
                if (kb == second && second > kb0) store_part(2 * wave);
            });
        if (second == kb1 && second > kb0) store_part(2 * wave);   // (an empty second part: 3 or 5 blocks in all)
        store_part(2 * wave + 1);
        __syncthreads();
        if (wave < NTB) {                                    // the wave's row block, its parts in order
            f32x4_t g = *at(0, wave, 0), u = GATEUP ? *at(0, wave, 1) : f32x4_t{};
#pragma unroll
            for (int part = 1; part < 8; ++part) {
                g += *at(part, wave, 0);
                if (GATEUP) u += *at(part, wave, 1);
            }
            if (wave * 16 + l16 < ti.rows)
                store_unit<GATEUP>(j.out, (size_t)(ti.row0 + wave * 16 + l16) * features + unit * 16 + kq * 4, g, u);
        }
        __syncthreads();
    };
    const int row_end = ti.row0 + ti.rows;
    for (; ti.row0 < row_end; ti.row0 += 16 * MAXB) {
        ti.rows = min(16 * MAXB, row_end - ti.row0);
        if constexpr (MAXB == 1) {
            body(IntTag<1>{});
        } else {
            const int ntb = (ti.rows + 15) >> 4;
            if (ntb <= 1) body(IntTag<1>{});
            else if (ntb <= 2) body(IntTag<2>{});
            else body(IntTag<4>{});
        }
    }
}

// A unit of one job of a launch that may hold two, in the parts the job has in a launch of its own: the bits of its rows do not depend
// on the other job.  (A launch has eight waves only where every job takes eight parts.)
template <bool GATEUP, int NW, int MAXB, int REGS, typename RowOf>
__device__ __forceinline__ void stream_unit_of(const FfnJob& j, const TileInfo& tile, int unit, f32x4_t* red, RowOf row_of) {
    if constexpr (NW == 4) {
        if (j.parts == 8) {
            stream_unit_eight<GATEUP, (MAXB < 4 ? MAXB : 4), REGS>(j, tile, unit, red, row_of);
            return;
        }
    }
    stream_unit<GATEUP, NW, MAXB, REGS>(j, tile, unit, (f32x4_t(*)[2][64])red, row_of);
}

hipError_t launch_gateup_stream(const FfnArgs& a, const FfnArgs* shared, hipStream_t s);
hipError_t launch_down_stream(const FfnArgs& a, const FfnArgs* shared, hipStream_t s);

}  // namespace lexi
