// Host-side launch of the query stage: picks the kernel variant for (d, d_bin, K).
#pragma once
#include "fg_query.hpp"
#include "fg_query_tile.hpp"
#include "fg_query_list.hpp"
#include "fg_query_leaf.hpp"
#include "fg_group_boxes.hpp"

namespace fg {

// ---- tile order: heaviest tiles first --------------------------------------------------------
// Tiles differ in cost by more than an order of magnitude (a tile inside a dense cluster scans thousands of
// candidates per query) and the hardware hands out workgroups in index order, so a heavy tile that starts late
// sets the kernel's end: measured on the 1M-point clustered workload the tile kernel took 1.2 ms for 0.73 ms of
// evenly spread work, the last third of it with most of the chip idle.  The tiles are therefore ranked by an
// estimate of their work, in 64 classes of half a power of two, heaviest class first.
// tile_order: [0, T) the order, [T, 2T) class of each tile (bit 6: uneven, see k_tile_work), [2T, 2T+64) class
// histogram, [2T+64, 2T+128) cursors.  The histogram is zero between calls: the binning clears it, and k_list_compact, the
// first kernel that nothing follows that reads it, does again (a launch of its own to clear it took 4 us of every call); should a
// call have ended between the two, k_tile_rank sees that it counts too many tiles.  The cursors are cleared by k_tile_work.

// The work list of the list kernel from the tiles' hand-over marks: blocks of 1024 tiles, the queries of a block in
// tile order (a block's place in the list comes from one atomic add, so blocks may swap, 65 536 queries each).
static __global__ void __launch_bounds__(1024) k_list_compact(const uint64_t* __restrict__ handed, int32_t n_tiles,
                                                              int32_t* __restrict__ work_list, int32_t* __restrict__ work_count,
                                                              int32_t* __restrict__ tile_counters /* to be cleared, or nullptr */)
{
    if (tile_counters && blockIdx.x == 0 && threadIdx.x < 2 * kTileClasses) tile_counters[threadIdx.x] = 0;
    __shared__ int32_t wave_tot[16];
    __shared__ int32_t block_base;
    const int32_t t = blockIdx.x * 1024 + threadIdx.x;
    const uint64_t m = t < n_tiles ? handed[t] : 0ull;
    const int32_t c = __popcll(m);
    int32_t incl = c;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    if (lane == 63) wave_tot[wv] = incl;
    __syncthreads();
    int32_t before = 0, total = 0;
    for (int j = 0; j < 16; ++j) {
        const int32_t w = wave_tot[j];
        if (j < wv) before += w;
        total += w;
    }
    if (threadIdx.x == 0) block_base = total > 0 ? atomicAdd(work_count, total) : 0;
    __syncthreads();
    int32_t at = block_base + before + incl - c;
    for (uint64_t rest = m; rest; rest &= rest - 1)
        work_list[at++] = t * kQueryBlock + (__ffsll((unsigned long long)rest) - 1);
}

__device__ __forceinline__ int32_t tile_class(int32_t work)
{
    if (work < 2) return work < 1 ? 0 : 1;
    const int32_t lg = 31 - __clz(work);
    const int32_t c = 2 * lg + ((work >> (lg - 1)) & 1);
    return c < kTileClasses ? c : kTileClasses - 1;
}

constexpr int kTilesPerWave = 16, kTilesPerWaveFew = 8;      // the second up to kFewTiles tiles: one round of the chain of loads instead of two
constexpr int kFewTiles = 8192;
// How many tiles, the first of the order, another kernel takes: those of dense_class and above, or, with all_from > 0, all if so many
// are of it, else none.
struct TileShare {
    int32_t dense_class, all_from;
    int32_t* n_dense;                             // nullptr: not asked, and dense_class is 0 or (no class) 64
    __device__ void write(int32_t m, int32_t n_tiles) const
    {
        if (n_dense) *n_dense = all_from == 0 ? m : (m >= all_from ? n_tiles : 0);
    }
};

// Work estimate of a tile: what the first two shells cost it without any pruning, i.e. for every column of the
// 3 x ... x 3 neighbourhood the longest candidate run any of its queries has there (the tile kernel scans a
// column for as long as its busiest lane needs), summed over the columns.  Taken over 8 of the tile's 64 queries
// (every ninth: consecutive queries mostly share their bins), 8 tiles per wavefront at a time: with all 64 the
// gathers of the bin boundaries made this kernel cost 73 us per million points.
constexpr int kTileSamples = 8;
constexpr int kFlatLaneUsePct = 60;   // below this estimated lane use (per cent) a tile takes the flattened scan
static_assert(kTileClasses == (1 << kTileFlatBit), "the flag sits above the class bits");

// maximum / sum over each aligned group of 8 lanes, returned in all 8 (DPP: swap inside pairs, swap pairs, mirror the half row)
__device__ __forceinline__ int32_t oct_max_i32(int32_t v)
{
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0xb1, 0xf, 0xf, false));    // quad_perm [1,0,3,2]
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x4e, 0xf, 0xf, false));    // quad_perm [2,3,0,1]
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false));   // row_half_mirror
    return v;
}
__device__ __forceinline__ int32_t oct_sum_i32(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(v, v, 0xb1, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(v, v, 0x4e, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false);
    return v;
}

// Where the group kernel may serve the call, the blocks behind the first `blocks` make its boxes
// (of its leaves, those of k_tile_rank of its nodes; ranking the tiles here, too, by the last block to finish, took longer than the launch
// that it saves: 100k points 18 us against 7 and 7).
template <int D, int DB>
static __global__ void __launch_bounds__(256) k_tile_work(QueryArgs a, int32_t n_tiles, int32_t blocks, int32_t tiles_per_wave)
{
    if constexpr (D <= kClustersMaxD) {
        if ((int32_t)blockIdx.x >= blocks) {
            const GroupTree tree = group_tree<D>(a.work_list, a.n);
            const int32_t leaf = ((int32_t)blockIdx.x - blocks) * 4 + (threadIdx.x >> 6);
            if (leaf < tree.n_leaf) group_leaf_box<D>(a.rec, a.n, tree, leaf);
            return;
        }
    }
    __shared__ int32_t hist[kTileClasses];
    if (threadIdx.x < kTileClasses) {
        hist[threadIdx.x] = 0;
        if (blockIdx.x == 0 && !a.votes) a.tile_order[2 * n_tiles + kTileClasses + threadIdx.x] = 0;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int sample = lane & (kTileSamples - 1);
    const int32_t wave_t0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * tiles_per_wave;
    int32_t ncols = 1;
#pragma unroll
    for (int c = 0; c < DB - 1; ++c) ncols *= 3;
    for (int32_t tb = wave_t0; tb < wave_t0 + tiles_per_wave; tb += kQueryBlock / kTileSamples) {
        const int32_t t = tb + (lane >> 3);
        const int32_t p = t * kQueryBlock + sample * 9;            // queries 0, 9, ..., 63 of the tile
        const bool live = t < n_tiles && p < a.n;
        int32_t cc[DB], seg_cell0 = 0;
        {
            const int32_t row = live ? __float_as_int(reinterpret_cast<const float*>(a.rec)[(int64_t)p * (rec_vecs(a.d) * 4) + a.d]) : 0;
            const int32_t b = live ? a.bin_idx[row] : 0;
            int32_t r = b % a.cells_per_segment;
            seg_cell0 = b - r;
            // the flat number counts slices of the last dimension (2^sub_shift per bin)
            const int32_t nz = a.n_bins << a.sub_shift;
            cc[DB - 1] = (r % nz) >> a.sub_shift;
            r /= nz;
#pragma unroll
            for (int c = DB - 2; c >= 0; --c) { cc[c] = r % a.n_bins; r /= a.n_bins; }
        }
        int32_t work = 0, around = 0, longest = 0, total = 0;
        for (int32_t col = 0; col < ncols; ++col) {
            int32_t rem = col, flat = 0;
            bool ok = live;
#pragma unroll
            for (int c = 0; c < DB - 1; ++c) {     // digit c of col -> offset -1, 0, +1 in dimension c
                const int32_t j = cc[c] + rem % 3 - 1;
                rem /= 3;
                ok = ok && j >= 0 && j < a.n_bins;
                flat = flat * a.n_bins + j;
            }
            int32_t len = 0;
            if (ok) {
                const int32_t cz = cc[DB - 1];
                const int32_t za = cz > 0 ? cz - 1 : 0, zb = cz < a.n_bins - 1 ? cz + 1 : a.n_bins - 1;
                const int32_t row = flat * a.n_bins;
                len = a.bounds[seg_cell0 + ((row + zb + 1) << a.sub_shift)] - a.bounds[seg_cell0 + ((row + za) << a.sub_shift)];
            }
            around += len;
            const int32_t col_max = oct_max_i32(len);
            work += col_max >> 2;                  // in passes of four; keeps the sum small
            longest += col_max;
            total += oct_sum_i32(len);
        }
        // A query with few points around it will not be certified after shell 1 (the k-th neighbour of a query at
        // the centre of its bin lies inside the inscribed ball of the 3-bin cube, about a sixth of its volume, only
        // if the cube holds some 6 K points); where more such queries than the tile kernel hands over are expected,
        // the tile will go on to shell 2: 5 x ... x 5 columns of 5-bin runs.
        const bool lonely = live && around < 4 * (a.slot0 + a.k_list);
        const bool goes_on = oct_sum_i32(lonely ? 1 : 0) * (kQueryBlock / kTileSamples) > a.defer_lanes;
        if (__any(goes_on)) {
            int32_t ncols2 = 1;
#pragma unroll
            for (int c = 0; c < DB - 1; ++c) ncols2 *= 5;
            for (int32_t col = 0; col < ncols2; ++col) {
                int32_t rem = col, flat = 0;
                bool ok = lonely && goes_on;
#pragma unroll
                for (int c = 0; c < DB - 1; ++c) {
                    const int32_t j = cc[c] + rem % 5 - 2;
                    rem /= 5;
                    ok = ok && j >= 0 && j < a.n_bins;
                    flat = flat * a.n_bins + j;
                }
                int32_t len = 0;
                if (ok) {
                    const int32_t cz = cc[DB - 1];
                    const int32_t za = cz > 1 ? cz - 2 : 0, zb = cz < a.n_bins - 2 ? cz + 2 : a.n_bins - 1;
                    const int32_t row = flat * a.n_bins;
                    len = a.bounds[seg_cell0 + ((row + zb + 1) << a.sub_shift)] - a.bounds[seg_cell0 + ((row + za) << a.sub_shift)];
                }
                work += oct_max_i32(len) >> 2;
            }
        }
        if (sample == 0 && t < n_tiles) {
            const int32_t cls = tile_class(work);
            // Uneven tile: over these columns its queries' runs average less than kFlatLaneUsePct of the longest
            // one, so a direct scan (every column as long as its busiest lane) leaves most lanes idle and the
            // flattened scan, at about twice the cost per pass, still comes out ahead.  Pruning, which this
            // estimate does not see, only widens the spread.
            const bool uneven = total * 100 < longest * kTileSamples * kFlatLaneUsePct;
            a.tile_order[n_tiles + t] = cls | ((uneven ? 1 : 0) << kTileFlatBit);
            atomicAdd(&hist[cls], 1);
        }
    }
    __syncthreads();
    if (threadIdx.x < kTileClasses && hist[threadIdx.x] > 0) {
        if (!a.votes) atomicAdd(&a.tile_order[2 * n_tiles + threadIdx.x], hist[threadIdx.x]);
        else if ((int32_t)threadIdx.x >= a.dense_class) atomicAdd(const_cast<int32_t*>(a.votes), hist[threadIdx.x]);
    }
}

// Position of every tile: classes in descending order; inside a class roughly the bin order (blocks of 256
// consecutive tiles reserve their places with one atomic per class, and a block's tiles keep the order in which
// its waves arrive), so that tiles running at the same time still share their neighbourhoods in the L2 cache.
template <int D>
static __global__ void __launch_bounds__(256) k_tile_rank(int32_t* __restrict__ order, int32_t n_tiles, TileShare share, GroupTree tree)
{
    if constexpr (D <= kClustersMaxD) {
        const int32_t blocks = (n_tiles + 255) >> 8;
        if ((int32_t)blockIdx.x >= blocks) {
            const int32_t node = ((int32_t)blockIdx.x - blocks) * 4 + (threadIdx.x >> 6);
            if (node < tree.n_node) group_node_box<D>(tree, node);
            return;
        }
    }
    __shared__ int32_t local[kTileClasses];   // this block's tiles per class, then the block's first position in the class
    __shared__ int32_t first[kTileClasses];   // position of the class's first tile: all heavier classes before it
    __shared__ int32_t counted;               // tiles in the histogram: all of them, or it holds an unfinished call's, too
    const int32_t t = blockIdx.x * 256 + threadIdx.x;
    const int32_t word = t < n_tiles ? order[n_tiles + t] : 0;
    static_assert(kTileClasses == 64, "one class per lane of the first wavefront");
    if (threadIdx.x < kTileClasses) {
        local[threadIdx.x] = 0;
        const int32_t own = order[2 * n_tiles + threadIdx.x];
        int32_t s = own;                      // with the classes above
#pragma unroll
        for (int o = 1; o < kTileClasses; o <<= 1) {
            const int32_t up = __shfl_down(s, o, 64);
            s += (int32_t)threadIdx.x + o < kTileClasses ? up : 0;
        }
        first[threadIdx.x] = s - own;
        if (threadIdx.x == 0) counted = s;
        if (blockIdx.x == 0 && (int32_t)threadIdx.x == share.dense_class) share.write(s, n_tiles);
    }
    __syncthreads();
    if (counted != n_tiles) {                 // no places can be had from it: tiles as they come, none another kernel's
        if (t < n_tiles) order[t] = t;
        if (blockIdx.x == 0 && threadIdx.x == 0 && share.n_dense) *share.n_dense = 0;
        return;
    }
    int32_t mine = 0;
    const int32_t cls = word & (kTileClasses - 1), uneven = (word >> kTileFlatBit) & 1;
    if (t < n_tiles) mine = atomicAdd(&local[cls], 1);
    __syncthreads();
    if (threadIdx.x < kTileClasses && local[threadIdx.x] > 0)
        local[threadIdx.x] = atomicAdd(&order[2 * n_tiles + kTileClasses + threadIdx.x], local[threadIdx.x]);
    __syncthreads();
    if (t < n_tiles) order[first[cls] + local[cls] + mine] = t | (uneven << kOrderFlagBit);
}

template <typename K>
static void allow_lds(K kernel, size_t bytes)
{
    if (bytes > 48 * 1024) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Two dimensions, many points: tiles whose queries meet 2000 candidates and more in their first shells (class 18: 512 passes
// of four) lie in bins that hold far more than their share, and go to the leaf kernel, whose boxes prune there because the points of
// such bins are put in order when they are binned.  Bins are made for K points, so the class rises with K (two classes are a
// factor of two).  Whole training step of 5M points of strongly varying density, K = 16, tile kernel alone against both 18 -> 4.1 ms.
// Query stage of such points for class 14 / 16 / 18 / 20 / 22, in us: 1.1M points in one split, K = 8 909 / 889 / 577 / 579 / 585, K = 16 1257 / 1246 /
// 682 / 697 / 709, K = 32 1255 / 1020 / 945 / 967 / 1015; 2M in four, K = 16 1271 / 994 / 995 / 1042 / 1056; 5M in five, K = 8 2477 / 2309 / 2087 / 2105 /
// 2146, K = 16 2674 / 2427 / 2415 / 2462 / 2517.
// Where no tile qualifies the four launches cost some 10 us from 1M points on (6 at 200k): of a whole call on uniform
// points 3 % at 1M and 1 % at 4M, so the line lies at 2^20 (kDenseMinN).
constexpr int32_t kDenseClass = 18;
static inline int32_t dense_class_for(int32_t k_list)
{
    int32_t c = kDenseClass;
    for (float k = 19.0f; k < (float)(k_list + 1); k *= 1.4142136f) ++c;       // 16 neighbours and what rounds to them: class 18
    return c;
}

// Clusters: which of two kernels serves the whole call is decided on the device, from the work estimates (k_tile_rank).  In
// clusters the tile kernel's densest tiles set its end, at some 0.25 to 0.5 us for a pass of their estimate, and the group kernel,
// which has no such tiles, takes a time that hardly depends on the cloud.  The call is the group kernel's if one tile in 512
// (at least four) is of a class whose time alone is beyond that; a class is returned, 0: the tile kernel's whatever the cloud.
// Query stage, tile + list kernel against group kernel, in us (U uniform, M 50 Gaussian clusters, S showers, P density r^(-5/3)):
//   d = 2, K = 10: 100k U 56 / 120, P 1358 / 186; 700k P 5017 / 2012      K = 40: 700k P 6679 / 4975
//   d = 3, K = 10: 100k U 80 / 202, M 198 / 185, S 451 / 184; 150k M 203 / 272, S 381 / 254      K = 40: 100k U 157 / 267, M 397 / 247, S 411 / 230
//   d = 4, K = 10: 100k U 174 / 296, M 1020 / 279; 400k M 1931 / 1173      K = 40: 100k U 253 / 427, M 850 / 419; 250k M 1519 / 1237
//   d = 5, K = 10: 100k U 428 / 473, M 3770 / 377; 700k M 10205 / 4131      K = 40: 100k U 546 / 703, M 1594 / 503; 700k M 9042 / 6074
// (The dense tiles alone to the group kernel, the others to the tile kernel, one after the other: of 100k M, d = 4 no gain, each of
// the two has its own end.)
static inline int32_t clusters_class_for(int32_t n, int32_t d, int32_t k_list)
{
    struct Line { int32_t most; float ns, ns_k, us_pass; };     // largest n; ns a query of the group kernel and for each neighbour; us a pass of the tile kernel
    static constexpr Line kLine[kClustersMaxD + 1] = {{0, 0, 0, 1}, {0, 0, 0, 1}, {1 << 20, 2.0f, 0.02f, 0.25f}, {1 << 17, 1.8f, 0.017f, 0.55f},
                                                      {3 << 17, 2.5f, 0.045f, 0.5f}, {1 << 20, 4.4f, 0.07f, 0.45f}};
    const Line& l = kLine[d];
    if (n > l.most) return 0;
    // (and longer by the share that n is of 2^20: its workgroups take their groups in fixed turns, 900k P in 4 splits, K = 16 2270 / 2740)
    const float passes = (float)n * 1e-3f * (1.0f + (float)n * 9.5e-7f) * (l.ns + l.ns_k * (float)(k_list + 1)) / l.us_pass;
    int32_t c = 2;
    for (float mid = 2.4f; mid < passes && c < kTileClasses; ++c) mid = (c & 1 ? 1.0f : 1.5f) * 1.2f * (float)(1 << ((c + 1) >> 1));
    return c < kTileClasses ? c : 0;
}

// The queries handed over by the tile (or leaf) kernel: their work list, then the list kernel.
template <int D, int DB, bool COUNT>
static hipError_t launch_handed(const QueryArgs& a, hipStream_t stream)
{
    const int grid = (a.n + kQueryBlock - 1) / kQueryBlock;
    const bool last = a.slot0 + a.k_list >= a.k - 1;                  // pass of a long list
    int32_t* const counters = a.tile_order ? a.tile_order + 2 * grid : (a.votes ? const_cast<int32_t*>(a.votes) - kTileClasses : nullptr);
    FG_LAUNCH(k_list_compact, dim3((grid + 1023) / 1024), dim3(1024), 0, stream, a.handed, grid, a.work_list, a.work_count,
              last ? counters : nullptr);
    // one query per wavefront; four times the wave slots of the chip: the queries differ widely in cost, and with
    // more, shorter workgroups the hardware dispatcher evens them out (cursors in memory cost more than they gained)
    // (where the call may be the group kernel's and nothing is handed over, 8192: an empty launch of 32,768 takes 7.8 us, of 8192 3)
    const int list_most = D > kClustersMaxD && a.votes ? 8192 : 32768;
    const int list_grid = a.n < list_most ? a.n : list_most;
    FG_LAUNCH((k_query_list_wave<D, DB, COUNT>), dim3(list_grid), dim3(kQueryBlock), 0, stream, a);
    return hipSuccess;
}

// One pass of the fast path: tile kernel + list kernel for a.k_list <= 64 neighbours per query, or what takes their place.  The second
// pass of a long list (LOWER) keeps the order of the first, the choice made with it (a.dense_class) and, where the group kernel
// serves the call, its boxes: nothing is handed over then, so the work list that would take their place stays empty.
template <int D, int DB, bool COUNT, bool LOWER>
static hipError_t launch_query_pass(QueryArgs& a, hipStream_t stream)
{
    const int grid = (a.n + kQueryBlock - 1) / kQueryBlock;
    const bool leaf = D == 2 && takes_dense_order(a.n, D);             // the dense tiles the leaf kernel's
    int32_t* const order = a.tile_order;
    if (!LOWER && D <= kClustersMaxD && !COUNT && a.algo == 0 && a.bin_idx && (grid > 1024 || asks_votes(a.n, D, a.n_segments, a.k)))
        a.dense_class = leaf ? dense_class_for(a.k_list) : clusters_class_for(a.n, D, a.k_list);
    const bool ranked = a.bin_idx && grid > 1024;                      // else a few waves per SIMD: nothing to reorder
    const bool clusters = a.dense_class > 0 && !leaf;                  // all tiles the group kernel's, perhaps
    const int32_t all_from = clusters ? (grid < 2048 ? 4 : grid / 512) : 0;
    if (!LOWER && clusters && !ranked) {
        a.votes = order + 2 * grid + kTileClasses;                     // a cursor that nothing else uses then
        a.votes_for = all_from;
    }
    if (!LOWER && (ranked || clusters)) {
        const int per_wave = grid <= kFewTiles ? kTilesPerWaveFew : kTilesPerWave;
        const int blocks = (grid + 4 * per_wave - 1) / (4 * per_wave);
        const GroupTree tree = group_tree<D>(a.work_list, a.n);
        FG_LAUNCH((k_tile_work<D, DB>), dim3(blocks + (clusters ? (tree.n_leaf + 3) / 4 : 0)), dim3(256), 0, stream, a, grid,
                  blocks, per_wave);
        if (ranked) {
            const TileShare share{a.dense_class, all_from, a.dense_class > 0 ? a.work_count + 1 : nullptr};
            FG_LAUNCH(k_tile_rank<D>, dim3((grid + 255) / 256 + (clusters ? (tree.n_node + 3) / 4 : 0)), dim3(256), 0, stream, order,
                      grid, share, tree);
        }
    }
    if (!ranked) a.tile_order = nullptr;
    if (clusters) FG_TRY(launch_query_clusters(a, stream));
    if constexpr (D == 2 && !COUNT) {
        if (a.dense_class > 0 && leaf) FG_TRY((launch_leaf_pass<D, LOWER>(a, stream)));
    }
    const int32_t cap = a.k_list;
    if (cap <= 16) {
        const size_t lds = tile_sorted_lds_bytes<16, D>();
        FG_LAUNCH((k_query_tile_sorted<D, DB, 16, COUNT, LOWER>), dim3(grid), dim3(kQueryBlock), lds, stream, a);
    } else if (cap <= 32) {
        const size_t lds = tile_sorted_lds_bytes<32, D>();
        FG_LAUNCH((k_query_tile_sorted<D, DB, 32, COUNT, LOWER>), dim3(grid), dim3(kQueryBlock), lds, stream, a);
    } else if (cap <= 48) {
        const size_t lds = tile_sorted_lds_bytes<48, D>();
        FG_LAUNCH((k_query_tile_sorted<D, DB, 48, COUNT, LOWER>), dim3(grid), dim3(kQueryBlock), lds, stream, a);
    } else {
        const size_t lds = tile_sorted_lds_bytes<64, D>();
        FG_LAUNCH((k_query_tile_sorted<D, DB, 64, COUNT, LOWER>), dim3(grid), dim3(kQueryBlock), lds, stream, a);
    }
    return launch_handed<D, DB, COUNT>(a, stream);
}

// From this many dimensions on the leaf kernel is the default.  Query stage, tile + list kernel against leaf kernel, in ms:
//   uniform points, one split                                    50 Gaussian clusters, width 0.03
//   200k, d = 6, K = 40    3.62 against 1.85     5k, d = 6, K = 10    0.28 against 0.14     100k, d = 6, K = 60  1.03 against 0.81
//   400k, d = 6, K = 10    3.80 against 1.68     1M, d = 6, K = 40   13.0  against 8.5      4M, d = 6, K = 16   32.3  against 30.9
//   400k, d = 7, K = 16    6.2  against 4.2      500k, d = 8, K = 64 21.4  against 10.0     60k, d = 10, K = 40  7.4  against 1.3
// Below, on uniform points, bins of one shell leave a query few hundred candidates and the tile kernel's scan is cheap next to
// the leaf kernel's fixed cost per tile:
//   1M, d = 5, K = 40      3.3  against 4.8      100k, d = 5, K = 40  0.55 against 0.76     1M, d = 4, K = 40    1.4  against 2.8
//   20k, d = 4, K = 24     0.14 against 0.21     1M, d = 3, K = 32    0.39 against 1.22
// There the leaf kernel is ahead on clusters and on few points (100k in clusters, d = 4, K = 40 1.13 against 0.62, d = 5
// 1.16 against 0.70; 5k uniform, d = 5, K = 16 0.35 against 0.14), which no size tells from the others.
constexpr int kLeafMinD = 6;

// Lists of more than 64 neighbours (K - 1 up to 127) take two passes: the first finds the 64 nearest, the second
// the rest, counting only keys above the 64th (keys are unique, so the split is exact).  A sorted list of more
// than 64 keys does not fit the 256 architectural registers of a wavefront next to everything else: held partly
// in accumulation registers it ran at one wavefront per SIMD with a copy at every use, 2.8x slower per query at
// K = 70 than at K = 65.
template <int D, int DB, bool COUNT>
static hipError_t launch_query_impl(const QueryArgs& a_in, hipStream_t stream)
{
    QueryArgs a = a_in;
    if (a.algo == 1) {
        const int grid = (a.n + kQueryBlock - 1) / kQueryBlock;
        const size_t heap_bytes = (size_t)(a.k > 1 ? a.k - 1 : 1) * kQueryBlock * sizeof(uint64_t);
        allow_lds(k_query_shell<D, DB, COUNT>, heap_bytes);
        FG_LAUNCH((k_query_shell<D, DB, COUNT>), dim3(grid), dim3(kQueryBlock), heap_bytes, stream, a);
        return hipSuccess;
    }
    const int32_t cap = a.k - 1;
    a.slot0 = 0;
    a.k_list = cap < 64 ? cap : 64;
    if constexpr (!COUNT) {
        if (a.algo == 3 || (a.algo == 0 && D >= kLeafMinD)) {
            const bool either = a.algo == 0 && a.bin_idx && asks_crowd(a.n, D, a.n_segments, a.k, a.dir != nullptr);      // decided on the device
            if (either) {
                a.votes = a.work_count + (a.n_segments < 16 || a.k >= 36 || a.n <= kCrowdAcross[D] ? 3 : 2);
                a.votes_for = a.n / 64;
                if (a.dir && a.n <= group_kernel_line(a.n, D, a.n_segments, a.k)) {
                    FG_TRY(launch_ask_votes(a, a.votes, a.work_count + 4, stream));
                    a.votes = a.work_count + 4;
                }
            }
            FG_TRY((launch_leaf_pass<D, false>(a, stream)));
            if (a.dir) FG_TRY((launch_handed<D, DB, false>(a, stream)));
            if (cap > 64) {
                a.slot0 = 64;
                a.k_list = cap - 64;
                FG_TRY((launch_leaf_pass<D, true>(a, stream)));
                if (a.dir) FG_TRY((launch_handed<D, DB, false>(a, stream)));
            }
            return either ? launch_query_group(a, stream) : hipSuccess;
        }
    }
    FG_TRY((launch_query_pass<D, DB, COUNT, false>(a, stream)));
    if (cap > 64) {
        a.slot0 = 64;
        a.k_list = cap - 64;
        FG_TRY((launch_query_pass<D, DB, COUNT, true>(a, stream)));
    }
    return hipSuccess;
}

template <int D, int DB>
static hipError_t launch_query_shell(const QueryArgs& a, hipStream_t stream)
{
    return a.out_cand ? launch_query_impl<D, DB, true>(a, stream) : launch_query_impl<D, DB, false>(a, stream);
}

template <int D>
static hipError_t dispatch_query_dbin(const QueryArgs& a, int32_t d_bin, hipStream_t stream)
{
    switch (d_bin) {
        case 2: return launch_query_shell<D, 2>(a, stream);
        case 3: if constexpr (D >= 3) return launch_query_shell<D, 3>(a, stream); break;
        case 4: if constexpr (D >= 4) return launch_query_shell<D, 4>(a, stream); break;
        case 5: if constexpr (D >= 5) return launch_query_shell<D, 5>(a, stream); break;
        default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace fg
