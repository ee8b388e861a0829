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

template <int G>
__device__ __forceinline__ bool fetch_tile(const int32_t* sched, int tile, int M, int tile_rows, TileInfo& ti) {
    TileGroup g;
    if (!fetch_group<G>(sched, tile, M, tile_rows, g)) return false;
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
// The grid is 1-D: 8 * ceil(ncb * max_tiles / 8) workgroups, times ksplit.
constexpr int kCbGroup = 2;

// With ksplit > 1 every item appears ksplit times in a row, once per part of the reduction dimension.
template <int G>
__device__ __forceinline__ bool fetch_item(const int32_t* sched, int ncb, int M, int tile_rows, int ksplit, TileInfo& ti, int& cb,
                                           int& part) {
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
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

hipError_t launch_gateup_stream(const FfnArgs& a, hipStream_t s);
hipError_t launch_down_stream(const FfnArgs& a, hipStream_t s);

}  // namespace lexi
