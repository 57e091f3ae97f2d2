// Internal declarations shared by the translation units of libfastgraph_hip.so (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fastgraph.h"

namespace fg {

constexpr int kGeomStride = 4;   // floats per (segment, binning dim): lo, inv_w, w, slack
constexpr int kTileClasses = 64; // classes of a tile's work estimate: as many counters and cursors behind the order of the tiles
constexpr int kKeyStride = 16;   // words between two bounding-box keys: one 64-byte line each, so that the
                                 // atomics on different keys do not queue up behind one another in one L2 line

// Everything the query stage needs; plain device pointers.
struct QueryArgs {
    const float4* rec;         // [n][rec_vecs(d)] bin-ordered point records: coordinates, original row, padding
    const int32_t* bounds;     // [S*T+1], T counted in slices (see sub_shift)
    const float* geom;         // [S][d_bin][4]
    const int32_t* row_splits; // [S+1]
    const int32_t* dir;        // [n] direction flags in ORIGINAL row order, or nullptr
    int32_t* out_idx;          // [n][k]
    float* out_d2;             // [n][k]
    int32_t* out_cand;         // [n] or nullptr
    int32_t* work_list;        // [n] sorted positions of handed-over queries, in bin order; before that the leaf kernel's boxes
    int32_t* work_count;       // [5] queries on the work list; dense tiles (see dense_class); points of crowded cells, the same and n if a tile lies across splits; either and n if half of the points ask or few are neighbours
    uint64_t* handed;          // [ceil(n/64)] per tile: which of its 64 queries the tile (or leaf) kernel hands over
    const int32_t* bin_idx;    // [n] flat bin of each point, original row order
    int32_t* tile_order;       // [2*ceil(n/64) + 128]: tile order, tile classes, class histogram, class cursors
    int32_t n;
    int32_t d;                 // coordinates per point (the record length follows from it)
    int32_t n_segments;
    int32_t k;                 // slots per output row
    int32_t slot0;             // tile, list and leaf kernels: neighbours already placed by an earlier pass (0 or 64); this pass keeps only keys above the one in row slot `slot0`
    int32_t k_list;            // tile, list and leaf kernels: neighbours this pass finds (1..64, or 0 for K = 1); they go to row slots slot0+1 .. slot0+k_list
    int32_t n_bins;
    int32_t cells_per_segment; // T: bins of a row split times the slices per bin
    int32_t sub_shift;         // log2 of the slices every bin is cut into along the last binning dimension
    int32_t algo;              // 0: the default of the sizes, 1: one lane per query for everything, 2: tile + list kernel with the flattened scan on every tile, 3: leaf kernel, 4: tile + list kernel, 5: group kernel
    int32_t defer_lanes;       // tile kernel: go on past shell 1 only while more lanes than this are unfinished
    // of some kernels only, and last: the fields above keep their places in the other kernels' arguments
    int32_t dense_class;       // > 0: tiles of this work class and above decide which are not the tile kernel's (the first work_count[1] of the order)
    int32_t few_ask;           // leaf kernel: tiles of which no more queries than this ask (direction flags) are handed over
    const float* coords;       // [n][d] the points in their original order: given (and rec not) where nothing was binned, else nullptr
    const int32_t* votes;      // few tiles, which are not ranked: as many of them are of dense_class and above (d >= 6: points of crowded cells); votes_for and all are the group kernel's
    int32_t votes_for;
};

struct OrderArgs;

// A chain of launches ends at the first that fails: what follows would run on what that one has not written (counters not
// cleared, an order not made).
#define FG_TRY(call)                                            \
    do {                                                        \
        const hipError_t fg_try_ = (call);                      \
        if (fg_try_ != hipSuccess) return fg_try_;              \
    } while (0)
#define FG_LAUNCH(...)                                          \
    do {                                                        \
        hipLaunchKernelGGL(__VA_ARGS__);                        \
        FG_TRY(hipGetLastError());                              \
    } while (0)

// Host-side launchers, one per translation unit.  Each returns the error of its first launch that failed.
hipError_t launch_binning(const float* coords, const int32_t* row_splits, int32_t n, int32_t d,
                          int32_t n_segments, int32_t n_bins, int32_t d_bin, int32_t sub_shift /* last binning dimension:
                          n_bins << sub_shift slices */, int64_t total_bins,
                          uint32_t* bbox_keys, float* geom, int32_t* bin_idx, int32_t* rank,
                          int32_t* perm, float* rec, int32_t* bounds,
                          int32_t* scan_partials,
                          int32_t morton_bits /* 0: row-major bins, the bin-ordered point records written to rec (perm unused);
                                                 b > 0 (the backward's row order): n_bins = 2^b, bit-interleaved bin order,
                                                 only perm is written, plus for d = 3 a copy of coords in the original
                                                 order padded to float4 in place of the records */,
                          int32_t* tile_counters /* [2 * kTileClasses] of the query stage, cleared; nullptr with morton_bits */,
                          int32_t* crowd /* [2] for counts_crowd, else nullptr */,
                          const OrderArgs* order /* dense cells' points are put in order, nullptr: not */,
                          hipStream_t stream);

// Up to this many points and one list of keys (K <= 65) every pair is compared, one wavefront per query, without bins.
// Whole forward call, one split, against binning and the bins' kernels:
//   1000 points: d = 3, K = 10  70 -> 11 us; d = 5, K = 40 293 -> 15 us; d = 10, K = 20 122 -> 13 us
//   4000 points: d = 2, K = 16  53 -> 25 us; d = 3, K = 40 122 -> 35 us; d = 8, K = 64  327 -> 50 us
// The cost grows with the square of n and two-dimensional bins, the cheapest, meet it at some 6000 points.
constexpr int32_t kSmallN = 4096;
inline bool takes_small_path(int64_t n, int32_t k) { return n <= kSmallN && k <= 65; }

// Sizes up to which the group kernel (one wavefront for two or four queries) serves a call: it fills the chip from a few thousand
// points on, where the kernels of one wavefront for 64 queries have fewer wavefronts than SIMDs and the densest tile sets their
// end, but it does not share a query's candidates with 64 others.  The lines are those of uniform points, which suit the others
// best (up to 15 % beyond, where clusters would lose as much to the launches of a choice), and depend on K with the size of the tile kernel's lists (K = 16, 32 and 64, whose rows leave from its registers, are its best).
// Query stage, tile + list kernel or leaf kernel against the group kernel, in us, uniform points of one split:
//   d = 2, K = 10: 5k points 29 / 21, 10k 29 / 27, 16k 29 / 36 (the quicker binning of few points makes up for that); K = 24: 20k 46 / 41, 26k 46 / 50;
//     K = 32: 13k 36 / 34, 20k 38 / 42, 33k 40 / 56; K = 40: 26k 70 / 54, 33k 72 / 60; K = 64: 20k 63 / 54, 26k 63 / 64, 33k 65 / 72
//   d = 3, K = 10: 5k 44 / 25, 16k 45 / 46, 20k 47 / 53; K = 32: 16k 61 / 60, 20k 62 / 68, 41k 68 / 120; K = 40: 26k 102 / 89, 33k 104 / 107, 41k 109 / 125;
//     K = 64: 26k 106 / 101, 33k 107 / 122; K = 100: 41k 331 / 282
//   d = 4, K = 10: 30k 117 / 107, 41k 121 / 135; K = 32: 30k 151 / 146, 35k 139 / 165; K = 40: 35k 197 / 176, 41k 183 / 200; K = 100: 41k 620 / 472
//   d = 5, K = 10: 60k 349 / 313, 80k 386 / 413; K = 32: 50k 457 / 366, 60k 386 / 418; K = 40: 60k 536 / 454, 70k 488 / 511; K = 100: 80k 1423 / 1409
//   d = 6, K = 20: 41k 358 / 347; K = 64: 55k 847 / 716      d = 7, K = 20: 41k 523 / 503      d = 8, K = 20: 36k 565 / 559      d = 9, K = 20: 25k 493 / 478
//   d = 10, K = 20: 16k 412 / 381, 20k 430 / 453
// of 16 splits: d = 4, K = 32 50k 155 / 150, 65k 161 / 186; K = 40 65k 207 / 205; K = 100 65k 761 / 498; d = 5, K = 24 100k 486 / 376, 130k 471 / 506;
//   K = 40 130k 565 / 566, 180k 696 / 817; K = 100 130k 1572 / 1374; of 64: d = 4, K = 24 81k 206 / 163, 120k 193 / 249; d = 5, K = 24 140k 468 / 366, 180k 488 / 496.
// Clusters, where a tile's queries differ most, gain far beyond: 55k points in showers, d = 3, K = 9 437 / 81; 59k in a mixture, d = 6, K = 37 683 / 203; so
// above these lines the device decides where it can (asks_votes; from 65,537 points on always).  Of many splits in four and five dimensions it does not
// see them (mixture, 16 splits: d = 4, K = 10 70k 302 / 135; d = 5, K = 10 180k 1515 / 386, which estimates give to the tile kernel): there the
// lines lie where uniform points already lose a quarter.
// Splits of a few points (K < 24): up to five dimensions a grid of one bin, which the tile kernel scans for 64 queries at once, best
// where the lists fill; beyond, few leaves for a tile of many splits.  A group has two or four queries to share what it costs
// to start.  Query stage, the other kernels against the group kernel, in us:
//   10k points: d = 2, K = 10 6 points a split 17 / 20, 18 23 / 20; d = 3, K = 10 6 19 / 21, 12 30 / 21, K = 20 22 23 / 21; d = 4, K = 10 6 29 / 23, 12 18 / 23,
//   18 64 / 23; d = 5, K = 20 18 63 / 26, 27 24 / 27, 45 28 / 27, K = 16 40 169 / 26; d = 8, K = 16 5 27 / 31, 10 27 / 29
//   16k: d = 2, K = 10 12 22 / 25, K = 20 18 28 / 25; d = 3, K = 17 18 23 / 27, 22 39 / 27; d = 4, K = 17 12 34 / 29, 22 26 / 29, 27 77 / 31
//   30k: d = 4, K = 20 6 38 / 46, 27 29 / 45, 34 85 / 45; d = 5, K = 20 18 69 / 49, 27 29 / 48, 45 33 / 48; d = 6, K = 16 10 26 / 48, 40 38 / 45, 80 45 / 45
inline bool few_points_a_split(int64_t n, int32_t d, int32_t n_segments, int32_t k)
{
    static constexpr int32_t kOneBin[6] = {0, 0, 88, 110, 156, 244};     // percent of K: the automatic grid has one bin up to there
    if (k >= 24) return false;
    const int64_t splits = n_segments;
    const bool many = n > 12288;
    if (d >= 6) return n <= splits * (many ? 48 : 6);
    const bool fill = n >= splits * k;
    if (d <= 3 ? k > 17 && (d == 2 || !many) : !fill && (d == 5 || n <= 20480)) return false;
    const int32_t percent = d <= 3 && many && k >= 10 && k <= 17 ? 130 : kOneBin[d];      // (whole call, 20k points in splits of 11, d = 3, K = 10 85 / 98)
    return 100 * n <= splits * k * percent;
}

// Six dimensions and more: up to the first line the group kernel, beyond the second the leaf kernel, in between the leaf kernel only if
// the points are spread evenly and no tile lies across two splits, for the leaf kernel's slowest tile sets its end.  A tile of two distant
// parts takes twice as long, one in a cluster several times.  The scatter of the binning counts the points that find four times the
// mean and eight before them in their cell, of every eighth block: of 8 clouds from one Gaussian to 5000 clusters 1 to 90 %, of
// uniform points none.  Query stage, leaf kernel against group kernel, in us, K = 12 and 40:
//   45k, d = 6: uniform 406 / 379 and 556 / 509, one Gaussian 808 / 486 and 1208 / 666, 50 clusters 718 / 226 and 1638 / 293; K = 20 uniform 55k 452 / 536
//   61k, d = 6 in 16 splits of whole tiles: uniform 142 / 214 and 232 / 274, clusters 214 / 152 and 426 / 166; of 8 (61,111) uniform 1.2 times
//   50k, d = 7 in 16: uniform 150 / 202 and 222 / 249, clusters 232 / 140 and 362 / 149      61k, one split: uniform K = 10 678 / 763
//   49k, d = 8: uniform 768 / 817 and 979 / 1065, clusters 953 / 302 and 1726 / 374; in 16: uniform 142 / 221 and 234 / 271, clusters 235 / 145 and 513 / 159
//   30k, d = 9: uniform 610 / 580 and 758 / 744; 37k K = 20 0.88 times      29k, d = 10: uniform 587 / 664 and 704 / 830, clusters 821 / 224 and 1420 / 276
//   55k, d = 6, one split, K = 12: group kernel 0.88 times; K = 20 in 16 splits across tiles: 45k, d = 6 216 / 183 (whole call), 24k, d = 10 176 / 132
constexpr int32_t kCrowdTo[11] = {0, 0, 0, 0, 0, 0, 61440, 61440, 49152, 36864, 28672};
constexpr int32_t kCrowdAcross[11] = {0, 0, 0, 0, 0, 0, 52000, 46000, 40000, 34000, 28672};      // K < 36, 16 splits and more: beyond, tiles across splits do not count
inline int64_t crowd_from(int32_t d, int32_t n_segments, int32_t k)
{
    static constexpr int32_t kOne[3][5] = {{56000, 48000, 32000, 32000, 21000}, {44000, 44000, 30000, 26000, 20000}, {61440, 57000, 42000, 33000, 23000}};   // K up to 17, 35, more
    static constexpr int32_t kMany[2][5] = {{44000, 42000, 30000, 26000, 20000}, {57000, 55000, 42000, 33000, 23000}};
    if (n_segments == 1) return kOne[k <= 17 ? 0 : (k < 36 ? 1 : 2)][d - 6];
    return d >= 9 && k >= 36 && n_segments >= 12 ? kCrowdTo[d] : kMany[k < 36 ? 0 : 1][d - 6];
}
inline bool counts_crowd(int64_t n, int32_t d) { return d >= 6 && n > 20000 && n <= kCrowdTo[d]; }

inline int64_t group_kernel_line(int64_t n, int32_t d, int32_t n_segments, int32_t k)
{
    // by K: below 24, below 36, up to 65 (one list), more (two passes of the tile kernel)
    static constexpr int32_t kLine[4][6] = {{0, 0, 16384, 20480, 40960, 80000}, {0, 0, 28000, 25000, 37500, 72000},
                                            {0, 0, 32768, 35000, 40960, 76000}, {0, 0, 32768, 40960, 40960, 84000}};
    if (d >= 6) return crowd_from(d, n_segments, k);
    if (d >= 4 && n <= (int64_t)n_segments * 16384) return d == 4 ? 81920 : 180224;
    return kLine[k < 24 ? 0 : (k < 36 ? 1 : (k <= 65 ? 2 : 3))][d];
}
inline bool takes_group_kernel(int64_t n, int32_t d, int32_t n_segments, int32_t k)
{
    return n <= group_kernel_line(n, d, n_segments, k) && !few_points_a_split(n, d, n_segments, k);
}

// Few points: binned in one launch before the scatter (figures in fg_binning.hip), and the query stage asks for the tiles' votes.
constexpr int32_t kFewN = 49152;
inline bool few_points(int64_t n, int32_t d, int32_t n_segments) { return n <= kFewN && n * (d + 8) <= (int64_t)n_segments * 327680; }

// Up to 1024 tiles are not ranked.  Their estimates are made all the same, to vote whether the call is the group kernel's, where clusters are known
// to gain by it: for few points, and for some way beyond the group kernel's lines.  Two launches, 6 to 9 us of such a call's 60 to 400 on uniform
// points and 20 on clusters, which then take a third or a sixth of their time (30k points: mixture, d = 3, K = 12 275 / 130 us; showers in 16
// splits 570 / 86; 41k points, d = 3, K = 32: showers 583 / 171, uniform points 101 / 107, by the group kernel 143 and 153).  Elsewhere up to
// 65,536 points uniform calls would be 6 to 12 us slower, 8 % (60k, d = 2, K = 16 66 / 72; d = 4, K = 20 170 / 182); clusters would gain as much.
// In splits of less than kVotesSplit points nothing is dense: a tile's candidates are its splits' points (40k points, d = 3, K = 10 in
// splits of 20 99 / 107 us a call without and with the votes).
constexpr int32_t kVotesFrom = 16384, kVotesTo = 65536, kVotesSplit = 64;
inline bool asks_votes(int64_t n, int32_t d, int32_t n_segments, int32_t k)
{
    if (d > 5 || n <= kVotesFrom || n > kVotesTo || n < (int64_t)n_segments * kVotesSplit) return false;
    return few_points(n, d, n_segments) || (d == 3 && k >= 24 && n <= 40960) || (d == 4 && k >= 24 && n <= 40960);
}

// With direction flags below the lines, too, if fewer than half of the points ask (counted by a kernel of one workgroup; with few neighbours, too, the group kernel): the leaf kernel hands tiles of few
// queries to the list kernel.  Whole call, leaf and list against group kernel, uniform points, K = 24: 40k, d = 6, one in ten 153 / 240 us, three in
// ten 213 / 344, eight in ten 508 / 470; 30k, one in a hundred 135 / 155; 10k, one in ten 130 / 100; a mixture, 40k, one in ten 195 / 157.
inline bool asks_crowd(int64_t n, int32_t d, int32_t n_segments, int32_t k, bool dir)
{
    return counts_crowd(n, d) && (dir || n > group_kernel_line(n, d, n_segments, k)) && !few_points_a_split(n, d, n_segments, k);
}

// Two dimensions and many points: the densest tiles are the leaf kernel's (dense_class_for), and the points of dense cells are
// ordered for it when they are binned.  (Ordered in three to five dimensions, too, the kernels that search by boxes gained 0 to 5 %
// on clusters, and the sort took more.)
constexpr int64_t kDenseMinN = 1 << 20;
inline bool takes_dense_order(int64_t n, int32_t d) { return d == 2 && n > kDenseMinN; }

// d = 2..10, d_bin = 2..min(d,5)
hipError_t launch_query(const QueryArgs& a, int32_t d, int32_t d_bin, hipStream_t stream);

// the group kernel over all tiles in the order, if k_tile_rank gave them to it; up to kClustersMaxD dimensions, boxes are there
constexpr int kClustersMaxD = 5;
hipError_t launch_query_clusters(const QueryArgs& a, hipStream_t stream);

// every pair compared: takes_small_path
hipError_t launch_query_small(const QueryArgs& a, hipStream_t stream);

// votes, and n more where half of the points ask or few are neighbours (a.dir)
hipError_t launch_ask_votes(const QueryArgs& a, const int32_t* votes, int32_t* out, hipStream_t stream);

// the group kernel, whatever the size (with a.votes, if they say so)
hipError_t launch_query_group(const QueryArgs& a, hipStream_t stream);

// perm != nullptr: rows are taken in bin order (row of sorted position q = perm[q * perm_stride]: 1 for a plain
// permutation, the record length in words for the index field of the forward's point records) and combined in
// LDS; nullptr: plain atomic scatter.
// coords4 (d = 3 with perm only, else nullptr): coords padded to four floats per row.
hipError_t launch_backward(const float* grad_d2, const int32_t* idx, const float* coords, const float* coords4,
                           const int32_t* perm, int32_t perm_stride, int32_t n, int32_t d, int32_t k, float* grad_coords,
                           hipStream_t stream);

hipError_t launch_oc_helper(const int32_t* asso_idx, const int32_t* unique_idx, const int32_t* unique_rs_asso,
                            const int32_t* rs, int32_t n_vert, int32_t n_unique, int32_t n_splits, int32_t n_maxuq,
                            int32_t n_maxrs, int32_t calc_m_not, int32_t rot_block, int32_t* M, int32_t* M_not,
                            int32_t* counts /* workspace of oc_workspace_bytes(), or nullptr */, hipStream_t stream);
size_t oc_workspace_bytes(int64_t n_unique, int32_t n_maxrs);

// A bin-ordered point record: the d coordinates, then the original row index (its bits in a float), then zero
// padding up to a whole number of 16-byte vectors.  One scattered store per vector in the counting sort, one load
// per vector wherever a candidate is fetched.
constexpr int rec_vecs(int d) { return (d + 1 + 3) / 4; }
template <int D>
__device__ __forceinline__ void load_rec(const float4* __restrict__ rec, int64_t q, float (&x)[D], int32_t& row)
{
    constexpr int NV = rec_vecs(D);
    float w[NV * 4];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const float4 f = rec[q * NV + v];
        w[4 * v] = f.x; w[4 * v + 1] = f.y; w[4 * v + 2] = f.z; w[4 * v + 3] = f.w;
    }
#pragma unroll
    for (int c = 0; c < D; ++c) x[c] = w[c];
    row = __float_as_int(w[D]);
}
template <int D>
__device__ __forceinline__ int32_t rec_row(const float4* __restrict__ rec, int64_t q)
{
    return __float_as_int(reinterpret_cast<const float*>(rec)[q * (rec_vecs(D) * 4) + D]);
}

// Direction flags (paper Algorithm 2, useDir / dir[]): 0 or 2 = issues no query, 1 or 2 = is nobody's
// neighbour, anything else = both roles.
__device__ __forceinline__ bool dir_is_query(int32_t f) { return f != 0 && f != 2; }
__device__ __forceinline__ bool dir_is_neighbour(int32_t f) { return f != 1 && f != 2; }

// Key of an empty best-list slot: just above the bit pattern of +infinity, so every real key
// (finite or infinite squared distance) is below it and every NaN squared distance is not.
// Candidates excluded by a direction flag are staged with NaN coordinates and so can never be kept.
constexpr uint64_t kEmptyKey = 0x7f800001ull << 32;

// Segment of a (sorted or original) position: largest s with row_splits[s] <= p, skipping empty
// segments by construction (row_splits[s+1] > p).
__device__ __forceinline__ int32_t segment_of(const int32_t* __restrict__ row_splits,
                                              int32_t n_segments, int32_t p)
{
    int32_t lo = 0, hi = n_segments;   // invariant: row_splits[lo] <= p < row_splits[hi]
    while (hi - lo > 1) {
        int32_t mid = (lo + hi) >> 1;
        if (row_splits[mid] <= p) lo = mid; else hi = mid;
    }
    return lo;
}

// Bin index of coordinate x in one dimension.  Monotone non-decreasing in x, which is what the
// search's lower bounds rely on.
__device__ __forceinline__ int32_t cell_of(float x, float lo, float inv_w, int32_t n_bins)
{
    float t = (x - lo) * inv_w;
    int32_t c = (int32_t)floorf(t);
    c = c < 0 ? 0 : c;
    return c > n_bins - 1 ? n_bins - 1 : c;
}

}  // namespace fg
