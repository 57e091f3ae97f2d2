// Leaf kernel: one wavefront per tile of 64 consecutive bin-ordered queries, candidates filtered on the matrix cores.
//
// Same result as the tile kernel (paper Section 3, Algorithm 2: the exact K-1 best others by (distance, index));
// what differs is how unsearched points are ruled out and how candidates are sifted:
//   * the sorted points are cut into leaves of 32 consecutive points; every leaf, every 64 leaves and every 4096
//     leaves have the bounding box of their points over ALL d coordinates (k_leaf_boxes, k_node_boxes).  A tile
//     descends only where a box is near enough to one of its four groups of queries to improve a list there, by
//     the same lower bound that prunes bins elsewhere; 64 boxes are tested at a time, one per lane.  There are no
//     shells and nothing is handed over: when the descent ends, every point not looked at is strictly farther than
//     the k-th best of every query;
//   * two leaves (64 candidates) at a time are compared with all 64 queries by four v_mfma_f32_32x32x16_f16: the
//     matrix result's sign says whether a pair can matter (see LeafFilter).  The test errs only to the safe side, so
//     what passes is a superset of what the direct scan keeps;
//   * survivors are queued as positions per query in LDS; 16 at a time are fetched, their distance is computed in
//     float32 exactly as everywhere else, and sorted into the list in registers with the networks of fg_sortnet.hpp.
// What bounds it: vector issue, about 220 instructions per 64 x 64 pairs (40 conversion, 64 signs, 60 queueing; the four
// matrix instructions run beside other wavefronts' vector work) and some 1300 per merge of 16 survivors a lane at 64 keys,
// at two wavefronts per SIMD, which the list in registers allows.  Whole forward call against the tile kernel: 500k uniform
// points, d = 8, K = 64 21.5 -> 10.0 ms; 60k, d = 10, K = 40 7.0 -> 1.31 ms.
#pragma once
#include "fg_query_tile.hpp"

namespace fg {

constexpr int kLeafPts = 32;
constexpr int kDenseGrid = 16384;                   // most workgroups where only dense tiles are searched: there may be none (5M skewed
                                                    // points 13.5 ms with 8192, 13.3 with 32768; no dense tile among 4M: 8 and 16 us)
constexpr int kLeafTrig = 16;                       // queued survivors of a lane that start a merge
constexpr int kLeafQueue = kLeafTrig + kLeafPts;    // most a lane can hold: one block of 32 candidates on top of kLeafTrig - 1
// So many merges more than blocks, and blocks are compared exactly from then on; the second where every list holds nothing but
// copies of its query.  (Ordinary tiles take two merges a block for their own leaves, 4 to 6 blocks, and soon fewer than
// one for two.)
constexpr int kLeafSiftFrom = 24;
constexpr int kLeafSiftTies = 4;
constexpr int kLeafBigH = 60000;                    // filter value of a candidate that must not pass / a query that takes none
constexpr int kLeafAllT = -30000;                   // query term that lets every live candidate pass

// a node's box: D minima, D maxima, zero padding to whole 16-byte vectors
template <int D> constexpr int box_vecs() { return (2 * D + 3) / 4; }

struct LeafTree {
    float4* boxes;             // level 1, then level 2 and 3 where they exist
    int32_t n1, n2, n3;        // nodes per level
    bool has2, has3;           // a level is built only when the one below has more than 64 nodes
};

// Boxes live in the work list's area (4 bytes a point, at least 256 in all): level 1 takes up to 2.5 bytes a point
// (80 bytes per 32 points at d = 9, 10), the levels above a 64th of that; 80 * ceil(n / 32) <= max(256, 4 n) for
// every n, and with the upper levels, which need n > 2048, 80 * (n / 32 + 1) * (1 + 1/64 + 1/4096) + 160 <= 4 n.
static inline LeafTree leaf_tree(void* area, int32_t n)
{
    LeafTree t;
    t.boxes = reinterpret_cast<float4*>(area);
    t.n1 = (n + kLeafPts - 1) / kLeafPts;
    t.n2 = (t.n1 + 63) / 64;
    t.n3 = (t.n2 + 63) / 64;
    t.has2 = t.n1 > 64;
    t.has3 = t.n2 > 64;
    return t;
}

// |x - the coordinate of the lane below|; 0 in lane 0
__device__ __forceinline__ float leaf_step(float x)
{
    const int32_t v = __float_as_int(x);
    return fabsf(x - __int_as_float(__builtin_amdgcn_update_dpp(v, v, 0x138, 0xf, 0xf, false)));    // wave_shr:1
}

// the whole call is the group kernel's
template <int D> __device__ __forceinline__ bool leaf_not_asked(const QueryArgs& a) { return D > kClustersMaxD && a.votes && dense_tiles(a) > 0; }

template <int D>
static __global__ void __launch_bounds__(256) k_leaf_boxes(QueryArgs a, float4* __restrict__ boxes)
{
    const float4* __restrict__ rec = a.rec;
    const int32_t n = a.n;
    if (a.dense_class > 0 && dense_tiles(a) == 0) return;
    if (a.dense_class == 0 && blockIdx.x == 0 && threadIdx.x == 0) *a.work_count = 0;        // nothing is handed over on this path
    if (leaf_not_asked<D>(a)) return;
    for (int64_t p0 = (int64_t)blockIdx.x * 256; p0 < n; p0 += (int64_t)gridDim.x * 256) {
    const int32_t p = (int32_t)p0 + threadIdx.x;
    float x[D];
    int32_t row;
    load_rec<D>(rec, p < n ? p : n - 1, x, row);                     // past the end: the last point once more
    float mn[D], mx[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        mn[c] = x[c]; mx[c] = x[c];
#pragma unroll
        for (int o = 1; o < kLeafPts; o <<= 1) {
            mn[c] = fminf(mn[c], __shfl_xor(mn[c], o, 64));
            mx[c] = fmaxf(mx[c], __shfl_xor(mx[c], o, 64));
        }
    }
    if ((threadIdx.x & (kLeafPts - 1)) == 0 && p < n) {
        float w[box_vecs<D>() * 4] = {};
#pragma unroll
        for (int c = 0; c < D; ++c) { w[c] = mn[c]; w[D + c] = mx[c]; }
#pragma unroll
        for (int v = 0; v < box_vecs<D>(); ++v)
            boxes[(int64_t)(p / kLeafPts) * box_vecs<D>() + v] = make_float4(w[4 * v], w[4 * v + 1], w[4 * v + 2], w[4 * v + 3]);
    }
    }
}

template <int D>
__device__ __forceinline__ void load_box(const float4* __restrict__ boxes, int32_t node, float (&w)[box_vecs<D>() * 4])
{
#pragma unroll
    for (int v = 0; v < box_vecs<D>(); ++v) {
        const float4 f = boxes[(int64_t)node * box_vecs<D>() + v];
        w[4 * v] = f.x; w[4 * v + 1] = f.y; w[4 * v + 2] = f.z; w[4 * v + 3] = f.w;
    }
}

// box of 64 nodes of the level below, one wavefront each
template <int D>
static __global__ void __launch_bounds__(256) k_node_boxes(QueryArgs a, const float4* __restrict__ below, int32_t n_below, float4* __restrict__ boxes,
                                                           int32_t n_nodes)
{
    if ((a.dense_class > 0 && dense_tiles(a) == 0) || leaf_not_asked<D>(a)) return;
    const int32_t node = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (node >= n_nodes) return;
    const int32_t child = node * 64 + lane;
    float w[box_vecs<D>() * 4];
    load_box<D>(below, child < n_below ? child : n_below - 1, w);
#pragma unroll
    for (int c = 0; c < D; ++c) {
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            w[c] = fminf(w[c], __shfl_xor(w[c], o, 64));
            w[D + c] = fmaxf(w[D + c], __shfl_xor(w[D + c], o, 64));
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int v = 0; v < box_vecs<D>(); ++v)
            boxes[(int64_t)node * box_vecs<D>() + v] = make_float4(w[4 * v], w[4 * v + 1], w[4 * v + 2], w[4 * v + 3]);
    }
}

using half2_t = __fp16 __attribute__((ext_vector_type(2)));
using half8_t = _Float16 __attribute__((ext_vector_type(8)));
using acc16_t = float __attribute__((ext_vector_type(16)));

union HalfPack { half2_t h; uint32_t u; };
union Frag { uint32_t u[4]; half8_t h; };

__device__ __forceinline__ uint32_t pack_half(float a, float b)
{
    HalfPack p;
    p.h = __builtin_amdgcn_cvt_pkrtz(a, b);
    return p.u;
}
__device__ __forceinline__ float half_lo(uint32_t u) { HalfPack p; p.u = u; return (float)p.h.x; }
__device__ __forceinline__ float half_dot(uint32_t a, float acc)
{
    HalfPack p;
    p.u = a;
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(_Float16 __attribute__((ext_vector_type(2))), p.h),
                                  __builtin_bit_cast(_Float16 __attribute__((ext_vector_type(2))), p.h), acc, false);
}

// The sixteen half-precision words of a point for the pre-filter: D coordinates (relative to the tile's centre and
// scaled), then the two words `t0`, `t1` that sum to a scalar, then two words of the other side's scalar slots.
// A candidate carries (H hi, H lo, 1, 1), a query (1, 1, T hi, T lo) and its coordinates negated.
template <int D>
__device__ __forceinline__ void pack_slots(const float (&c)[D], float t0, float t1, float t2, float t3, uint32_t (&s)[8])
{
    float w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < D; ++i) w[i] = c[i];
    w[D] = t0; w[D + 1] = t1; w[D + 2] = t2; w[D + 3] = t3;
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = pack_half(w[2 * i], w[2 * i + 1]);
}
// half the squared norm of the coordinates as half precision holds them
template <int D>
__device__ __forceinline__ float half_norm(const float (&c)[D])
{
    float h = 0.0f;
#pragma unroll
    for (int i = 0; i < D; i += 2) h = half_dot(pack_half(c[i], i + 1 < D ? c[i + 1 < D ? i + 1 : i] : 0.0f), h);
    return 0.5f * h;
}

// maximum over the lanes up to and with the own one
__device__ __forceinline__ uint32_t wave_max_below(uint32_t v)
{
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0x111, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0x112, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0x114, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0x118, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0x142, 0xa, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, 0x143, 0xc, 0xf, false));
    return v;
}

// a value that is the same in all lanes, kept in a scalar register (the vector registers are what a long list is short of)
template <bool ON> __device__ __forceinline__ float uniform_value(float v) { return ON ? __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))) : v; }

// swaps the upper 32 lanes of a with the lower 32 lanes of b
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

template <int KC> constexpr int leaf_waves() { return KC <= 16 ? 3 : 2; }
template <int KC, int D> constexpr size_t leaf_lds_bytes()
{
    const size_t scan = (size_t)kLeafQueue * kQueryBlock * 4 + (size_t)(kQueryBlock * box_vecs<D>() * 4 + 4 * 2 * D + D + 2 * kQueryBlock) * 4;
    const size_t out = (size_t)kQueryBlock * 4 + (size_t)KC * kDumpStride * 4;
    return scan > out ? scan : out;
}

template <int D, int KC, bool LOWER>
__device__ __forceinline__ void leaf_tile(const QueryArgs& a, const LeafTree& tree, const int32_t tile, uint64_t* lds64)
{
    constexpr int NV = rec_vecs(D);
    constexpr int NB = box_vecs<D>();
    uint32_t* const queue = reinterpret_cast<uint32_t*>(lds64);                   // [kLeafQueue][64] sorted positions
    float4* const lbox = reinterpret_cast<float4*>(queue + kLeafQueue * kQueryBlock); // [64 nodes] boxes measured last
    float* const gbox = reinterpret_cast<float*>(lbox + kQueryBlock * NB);        // [4 groups][D minima, D maxima]
    float* const centre = gbox + 4 * 2 * D;                                       // [D] of the tile's box
    const int lane = threadIdx.x;
    const int32_t cap = a.k_list;
    const int32_t p = tile * kQueryBlock + lane;
    const int32_t pp = p < a.n ? p : a.n - 1;
    float x[D];
    int32_t my_row;
    load_rec<D>(a.rec, pp, x, my_row);
    const bool asks = !(a.dir && !dir_is_query(a.dir[my_row]));
    const bool valid = p < a.n;
    const int32_t seg = segment_of(a.row_splits, a.n_segments, pp);
    int32_t* const ends = reinterpret_cast<int32_t*>(centre + D);                 // [2][64] of the query's row split
    const int32_t sa = a.row_splits[seg], sb = a.row_splits[seg + 1];
    ends[lane] = sa;
    ends[kQueryBlock + lane] = sb;
    const int32_t pa = __builtin_amdgcn_readlane(sa, 0), pb = __builtin_amdgcn_readlane(sb, kQueryBlock - 1);
    const bool several = pa != __builtin_amdgcn_readlane(sa, kQueryBlock - 1);    // the tile spans several row splits
    // Where few queries ask they are handed to the list kernel, which gives each a wavefront, before any search.  Eight
    // neighbouring tiles decide together: one tile of many may have few by chance, or be the last, and would have the call wait
    // for its queries alone (d = 10: 0.17 ms).
    uint64_t few = 0;
    if (a.dir && a.dense_class == 0) {
        int32_t points = 0, ask = 0;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const int64_t pos = (int64_t)((tile & ~7) + b) * kQueryBlock + lane;
            const bool in = pos < a.n;
            points += __popcll(__ballot(in));
            ask += __popcll(__ballot(in && dir_is_query(a.dir[rec_row<D>(a.rec, in ? pos : 0)])));
        }
        if (cap > 0 && ask * kQueryBlock <= a.few_ask * points) few = __ballot(valid && asks);
        if (lane == 0) a.handed[tile] = few;
    }
    const bool active = valid && cap > 0 && asks && few == 0;
    uint64_t lower = 0;
    if (LOWER && active) {
        const int32_t li = a.out_idx[(int64_t)my_row * a.k + a.slot0];
        lower = li < 0 ? kEmptyKey : (((uint64_t)__float_as_uint(a.out_d2[(int64_t)my_row * a.k + a.slot0]) << 32) | (uint32_t)li);
    }
    uint64_t best[KC];
#pragma unroll
    for (int i = 0; i < KC; ++i) best[i] = (i < KC - cap) ? 0ull : kEmptyKey;
    uint32_t tau_hi = (uint32_t)(kEmptyKey >> 32);
    int32_t cnt = 0;

    if (__any(active)) {
    // The queries form four groups of consecutive ones, and boxes of points are tested against the groups' boxes.  The sorted
    // order runs along columns of bins and jumps at their ends; a group across a jump has a box that spans all
    // between, so the groups end at the three longest jumps (uniform points: about the columns that the tile spans).  Where
    // no jumps stand out, within a bin, they are 16 queries each.  (Always 16 each: 1M uniform points, d = 6, K = 8 7.8 ms, now 4.8;
    // 5000 clusters of 200 points, K = 16 2.9, now 1.45, with the tests of single queries on the upper level below.)
    int32_t g1 = 16, g2 = 32, g3 = 48;       // first queries of groups 1, 2, 3
    {
        float step = 0.0f;
#pragma unroll
        for (int c = 0; c < D && c < FG_MAX_D_BIN; ++c) step += leaf_step(x[c]);
        int32_t key = (__float_as_int(step) & ~63) | lane;
        const int32_t c0 = wave_max_i32(key);
        key = key == c0 ? 0 : key;
        const int32_t c1 = wave_max_i32(key);
        key = key == c1 ? 0 : key;
        const int32_t c2 = wave_max_i32(key);
        const float third = __int_as_float(c2 & ~63);       // (0 where the tile has but one or two steps)
        if (c0 >= kQueryBlock && __popcll(__ballot(step * 3.0f > third)) <= 16) {
            const int32_t l0 = c0 & 63, l1 = c1 & 63, l2 = c2 & 63;
            g1 = min(l0, min(l1, l2));
            g3 = max(l0, max(l1, l2));
            g2 = l0 + l1 + l2 - g1 - g3;
        }
    }
    // boxes of the four groups, and the tile's
    float hext = 0.0f;         // largest half extent of the tile
    float zmax = 0.0f;         // largest coordinate of its centre
    {
        // maximum from the lane's group's first query up to its own: what a step of the scan brings counts if it comes from there
        const int32_t start = lane >= g3 ? g3 : (lane >= g2 ? g2 : (lane >= g1 ? g1 : 0));
        const bool last = lane + 1 == g1 || lane + 1 == g2 || lane + 1 == g3 || lane == kQueryBlock - 1;
        const int32_t group = (lane >= g1) + (lane >= g2) + (lane >= g3);
        const bool in1 = lane - 1 >= start, in2 = lane - 2 >= start, in4 = lane - 4 >= start, in8 = lane - 8 >= start;
        const bool in_row = start < (lane & ~15), in_half = start < 32;
        auto group_max = [&](float v) __attribute__((always_inline)) -> float {
            const int32_t id = __float_as_int(-3.4028235e38f);
            auto from = [&](float t, bool in) __attribute__((always_inline)) { v = in ? fmaxf(v, t) : v; };
            from(__int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x111, 0xf, 0xf, false)), in1);
            from(__int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x112, 0xf, 0xf, false)), in2);
            from(__int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x114, 0xf, 0xf, false)), in4);
            from(__int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x118, 0xf, 0xf, false)), in8);
            from(__int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x142, 0xa, 0xf, false)), in_row);
            from(__int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x143, 0xc, 0xf, false)), in_half);
            return v;
        };
        auto over_groups = [&](float v) __attribute__((always_inline)) -> float {
            const int32_t w = __float_as_int(v);
            return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(w, g1 - 1)), __int_as_float(__builtin_amdgcn_readlane(w, g2 - 1))),
                         fmaxf(__int_as_float(__builtin_amdgcn_readlane(w, g3 - 1)), __int_as_float(__builtin_amdgcn_readlane(w, 63))));
        };
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const float mx = group_max(active ? x[c] : -3.4028235e38f), mn = -group_max(active ? -x[c] : -3.4028235e38f);
            if (last) { gbox[group * 2 * D + c] = mn; gbox[group * 2 * D + D + c] = mx; }
            const float tmx = over_groups(mx), tmn = -over_groups(-mn);
            const float zc = tmn * 0.5f + tmx * 0.5f;
            if (lane == 0) centre[c] = zc;
            hext = uniform_value<(KC > 48)>(fmaxf(hext, fmaxf(tmx - zc, zc - tmn)));
            zmax = uniform_value<(KC > 48)>(fmaxf(zmax, fabsf(zc)));
        }
    }
    __syncthreads();

    // ---- the pre-filter ----
    // Everything is taken relative to the tile's centre z and scaled by a power of two `scale` that puts the tile and
    // the reach of its lists inside [-32, 32]; candidates are clamped to that cube (which holds every query, so a
    // clamped candidate only comes nearer).  Let q', c' be these points and q, c their half-precision roundings
    // (towards zero: 2^-10 relative, 2^-14 where denormals are flushed).  A candidate that can enter the list has
    // |q' - c'| <= rho', hence |c'| <= |q'| + rho' and by the triangle inequality
    //   |q - c| <= rho' + |q - q'| + |c - c'| <= rho' + 2^-10 (2 |q'| + rho') + 2 sqrt(10) 2^-14 =: r.
    // The matrix instruction forms  F = H + T - q.c  with H = |c|^2 / 2 and T = (|q|^2 - r^2) / 2 - slack, each as the
    // sum of two halves: F < 0 for every such candidate.  Products of halves are exact in float32; sixteen float32
    // additions of terms below |q|^2 + |c|^2 + r^2 <= 3 (|q| + r)^2 err by less than 2^-17 (|q| + r)^2, the halves of
    // H and T by 2^-20 relative or 2^-14 absolute each: slack = 2^-15 (|q| + r)^2 + 2^-11 covers both.
    // rho' comes from the k-th best distance, enlarged by 2^-15 for the rounding of distances and of the scaled
    // points; below 1e-30 (where squares lose their relative accuracy) 1e-30 stands in.  A list that is not full, or
    // whose k-th best is infinite, takes everything.
    float scale = 0.0f, zs[D];
    Frag b0, b1;                       // queries 0..31 and 32..63
    int32_t gtau[4];                   // per group: bits of the largest k-th best distance, -1: no query searches
    auto refresh = [&]() __attribute__((always_inline)) {
        const bool full = tau_hi < 0x7f800000u;
        const float rho = sqrtf(fmaxf(__uint_as_float(tau_hi), 1e-30f)) * 1.000031f;
        // with the group's number on top the maximum up to a group's last query is the group's (the two bits this takes are
        // rounded up)
        const uint32_t gm = wave_max_below((uint32_t)((lane >= g1) + (lane >= g2) + (lane >= g3)) << 29 | (active ? (tau_hi >> 2) + 1 : 0u));
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int32_t m = __builtin_amdgcn_readlane((int32_t)gm, g == 0 ? g1 - 1 : (g == 1 ? g2 - 1 : (g == 2 ? g3 - 1 : 63))) & 0x1fffffff;
            gtau[g] = m > 0 ? m << 2 : -1;
        }
        const int32_t rb = wave_max_i32(active && full ? __float_as_int(rho) : 0);
        // (not finer than the spacing of floats at the centre: a lone point has no extent, and a scale without bound would
        // overflow the scaled centre)
        const float reach = fmaxf(hext + __int_as_float(rb), zmax * 5.9604645e-8f);
        int32_t se = 258 - (int32_t)(__float_as_uint(reach) >> 23);     // reach < 2^(e - 126): scale * reach < 32
        se = se > 254 ? 254 : (se < 1 ? 1 : se);
        scale = uniform_value<(KC > 48)>(__int_as_float(se << 23));
        float q[D];
        float n2 = 0.0f;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            zs[c] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(centre[c] * scale)));
            q[c] = active ? __builtin_fmaf(x[c], scale, -zs[c]) : 0.0f;
            n2 = __builtin_fmaf(q[c], q[c], n2);
            q[c] = -q[c];
        }
        const float qn = sqrtf(n2) * 1.0001f;
        const float rs = rho * scale;
        const float r = rs + 0.000985f * (2.0f * qn + rs) + 0.0005f;
        const float s = qn + r;
        float t = half_norm<D>(q) - 0.5f * r * r - 3.06e-5f * s * s - 0.0005f;
        t = full ? t : (float)kLeafAllT;
        // a reach beyond the scale (only where the exponent was clamped) takes everything, too
        if (full && !(t > (float)kLeafAllT)) t = (float)kLeafAllT;
        t = active ? t : (float)kLeafBigH;
        const float th = half_lo(pack_half(t, 0.0f));
        uint32_t w[8];
        pack_slots<D>(q, 1.0f, 1.0f, th, t - th, w);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b0.u[i] = w[i];
            b1.u[i] = w[i + 4];
            swap_halves(b0.u[i], b1.u[i]);
        }
    };
    refresh();

    // ---- merging queued survivors ----
    constexpr int kFetch = NV == 1 || (NV == 2 && KC <= 48) ? 8 : 4;              // records requested together
    auto absorb = [&]() __attribute__((always_inline)) {
        uint64_t pend[kPend];
#pragma unroll
        for (int i0 = 0; i0 < kPend; i0 += kFetch) {
            int32_t pos[kFetch];
            float y[kFetch][D];
            int32_t src[kFetch];
#pragma unroll
            for (int i = 0; i < kFetch; ++i) {
                const int32_t at = cnt - 1 - (i0 + i);
                const int32_t in_queue = (int32_t)queue[(at >= 0 ? at : 0) * kQueryBlock + lane];
                pos[i] = at >= 0 ? in_queue : pp;
            }
#pragma unroll
            for (int i = 0; i < kFetch; ++i) load_rec<D>(a.rec, pos[i], y[i], src[i]);
#pragma unroll
            for (int i = 0; i < kFetch; ++i) {
                float diff = x[0] - y[i][0];
                float d2 = diff * diff;
#pragma unroll
                for (int c = 1; c < D; ++c) {
                    diff = x[c] - y[i][c];
                    d2 = d2 + diff * diff;
                }
                uint64_t key = ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)src[i];
                if (LOWER) key = key > lower ? key : kEmptyKey;
                key = pos[i] == pp ? kEmptyKey : key;               // the query itself, and empty places
                // the key is formed here: left to the compiler it is formed where the sort uses it, with all sixteen
                // records held in registers until then (100 to 200 spilled registers at d >= 8)
                asm volatile("" : "+v"(key));
                pend[i0 + i] = key;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        cnt = cnt > kPend ? cnt - kPend : 0;
        net_sort<kPend>(pend);
        net_absorb<KC, kPend>(best, pend);
        tau_hi = (uint32_t)(best[KC - 1] >> 32);
        refresh();
    };

    // ---- candidates that the filter does not tell apart ----
    // The filter's grain is a 2^-10 of the tile's extent.  Where it lets through more than that sorts out (equal points, two
    // dense clusters in one tile, an outlier's tile, far from all of which the k-th best differ by less than the grain), the
    // merges outnumber the blocks of 32 candidates: 746 merges against 40 in other tiles, 200k points in 50 clusters of width
    // 0.001, d = 8, K = 64.  From then on a block's survivors are compared with the k-th best, exactly and for all queries at
    // once, before they are queued: some 900 instructions for 32, less than one merge of 16.  Those points 3.5 -> 2.3 ms; 60k
    // points of which one in a thousand lies a thousand times as far out, d = 10, K = 64 16.1 -> 8 ms.
    int32_t excess = 0;                          // merges less blocks
    bool exact = false;
    auto sift = [&](int32_t base, uint32_t m) __attribute__((always_inline)) -> uint32_t {
        uint32_t keep = 0;
        float w[D];                              // the candidate of the lane's number
        int32_t from;
        load_rec<D>(a.rec, min(base + (lane & (kLeafPts - 1)), a.n - 1), w, from);
#pragma unroll 2
        for (int c = 0; c < kLeafPts; ++c) {
            float diff = x[0] - __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w[0]), c));
            float d2 = diff * diff;
#pragma unroll
            for (int i = 1; i < D; ++i) {
                diff = x[i] - __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w[i]), c));
                d2 = d2 + diff * diff;
            }
            const uint64_t key = ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)__builtin_amdgcn_readlane(from, c);
            keep |= (key < best[KC - 1] ? 1u : 0u) << c;
        }
        return m & keep;
    };

    // ---- 64 candidates against 64 queries ----
    // matrix row r of a block of 32 carries candidate 16 * (r >> 2 & 1) + 4 * (r >> 3) + (r & 3), so that the 16 signs of
    // a lane and the 16 of its partner half are the candidates in order
    const int32_t my_cand = ((lane >> 2) & 1) * 16 + (((lane & 31) >> 3) << 2) + (lane & 3);
    struct Raw { float4 v[NV]; int32_t leaf0, leaf1; bool live; };
    auto fetch = [&](int32_t leaf0, int32_t leaf1) __attribute__((always_inline)) -> Raw {
        Raw r;
        r.leaf0 = leaf0; r.leaf1 = leaf1;
        const int32_t q = (lane < 32 ? leaf0 : leaf1) * kLeafPts + my_cand;
        r.live = q >= pa && q < pb && (lane < 32 || leaf1 >= 0);
        const int64_t at = r.live ? q : pp;
#pragma unroll
        for (int v = 0; v < NV; ++v) r.v[v] = a.rec[at * NV + v];
        return r;
    };
    auto signs = [&](const acc16_t& f) __attribute__((always_inline)) -> uint32_t {
        uint32_t m = 0;
#pragma unroll
        for (int v = 15; v >= 0; --v) m = __builtin_amdgcn_alignbit(m, __float_as_uint(f[v]), 31);
        return m;
    };
    // ---- which leaves ----
    const int32_t la = pa / kLeafPts, lb = (pb + kLeafPts - 1) / kLeafPts;        // leaves of the tile's row splits
    // first the tile's own leaves, with one more on either side for long lists: they fill the lists
    const int32_t around = cap > 16 ? 2 : 1;
    const int32_t own_a = tile * 2 - around, own_b = tile * 2 + 1 + around;       // inclusive
    float b2[4];
    // squared lower bounds between this lane's box and the four groups' boxes
    auto measure = [&](const float4* __restrict__ boxes, int32_t node) __attribute__((always_inline)) {
        float w[NB * 4];
        load_box<D>(boxes, node, w);
        asm volatile("" ::: "memory");      // the groups' boxes are read here, not kept in 8 D registers across the search
#pragma unroll
        for (int v = 0; v < NB; ++v) lbox[lane * NB + v] = make_float4(w[4 * v], w[4 * v + 1], w[4 * v + 2], w[4 * v + 3]);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            float s = 0.0f;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const float gap = fmaxf(fmaxf(w[c] - gbox[g * 2 * D + D + c], gbox[g * 2 * D + c] - w[D + c]), 0.0f);
                s = c == 0 ? gap * gap : s + gap * gap;
            }
            b2[g] = s;
            __builtin_amdgcn_sched_barrier(0);      // one group's box in registers at a time
        }
    };
    // can a point of the measured box enter a list of one of the groups
    auto reaches = [&]() __attribute__((always_inline)) -> bool {
        bool hit = false;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const bool out = gtau[g] < 0 || (gtau[g] < 0x7f800000 && b2[g] > 1e-30f && __int_as_float(gtau[g]) < b2[g] * kBoundShrink);
            hit = hit || !out;
        }
        return hit;
    };
    float near_limit[4];
    auto near = [&]() __attribute__((always_inline)) -> bool {
        return b2[0] <= near_limit[0] || b2[1] <= near_limit[1] || b2[2] <= near_limit[2] || b2[3] <= near_limit[3];
    };
    const float4* const box1 = tree.boxes;
    const float4* const box2 = box1 + (int64_t)tree.n1 * NB;
    const float4* const box3 = box2 + (int64_t)tree.n2 * NB;
    const int32_t l_last = lb - 1;
    // Sweep 0 takes the tile's own leaves; sweep 1 the boxes within an eighth of the distance the lists reach after
    // that; sweep 2 the rest, with lists that have tightened by then (500k uniform points, d = 8, K = 64,
    // with groups of 16: 12.2 ms; within a quarter 12.6, a half 14.9, without sweep 1 21.1; two or three rings 12.5 to 13.1).  m3, m2, m1: nodes of the
    // current 64 of each level still to be taken.
    int32_t sweep = 0, t3 = (l_last >> 12) + 1, first3 = 0, first2 = 0, first1 = own_a;
    uint64_t m3 = 0, m2 = 0, m1 = 0;
    for (int32_t l = own_a; l <= own_b; ++l) if (l >= la && l <= l_last) m1 |= 1ull << (l - own_a);
#pragma unroll
    for (int g = 0; g < 4; ++g) { b2[g] = 0.0f; near_limit[g] = 0.0f; }
    // A group's box is often much larger than the reach of its queries (a run of the sorted order that wraps from the end
    // of one column of bins to the next, an isolated point among close ones): the nodes that the groups let through are
    // tested once more against every query by itself, the leaves and the nodes above (on the leaves alone, a tile at the wrap
    // of the first dimensions tested them all, and a handful of such tiles took the kernel's time: 200k points on a lattice of
    // 4^6, K = 16 0.98 ms, now 0.19).
    // Of the leaves under a node every eighth is tested first; where that drops less than a third (from d = 8 on nearly every
    // box reaches), the others are left out, and so is the next node, then the next three, seven, and so on up to 63.
    int32_t wait = 0, pause = 0;
    constexpr uint64_t kProbe = 0x0101010101010101ull;
    auto each_query = [&](uint64_t m, uint64_t which) __attribute__((always_inline)) -> uint64_t {
        __syncthreads();
        for (uint64_t mm = which; mm;) {             // two at a time: one alone is a chain of some 450 clocks
            int j[2];
            j[0] = __builtin_ctzll(mm);
            mm &= mm - 1;
            j[1] = mm ? __builtin_ctzll(mm) : j[0];
            mm &= mm - 1;
            float w[2][NB * 4], s[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < NB; ++v) {
                    const float4 f = lbox[j[i] * NB + v];
                    w[i][4 * v] = f.x; w[i][4 * v + 1] = f.y; w[i][4 * v + 2] = f.z; w[i][4 * v + 3] = f.w;
                }
#pragma unroll
            for (int c = 0; c < D; ++c) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const float gap = fmaxf(fmaxf(w[i][c] - x[c], x[c] - w[i][D + c]), 0.0f);
                    s[i] = c == 0 ? gap * gap : s[i] + gap * gap;
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const bool out = !active || (tau_hi < 0x7f800000u && s[i] > 1e-30f && __uint_as_float(tau_hi) < s[i] * kBoundShrink);
                if (!__any(!out)) m &= ~(1ull << j[i]);
            }
        }
        __syncthreads();
        return m;
    };
    // fills m1 with leaves to visit; false: the sweep is over
    auto advance = [&]() __attribute__((always_inline)) -> bool {
        while (!m1) {
            if (m2) {
                first1 = (first2 + __builtin_ctzll(m2)) << 6;
                m2 &= m2 - 1;
                const int32_t n1 = first1 + lane;
                const bool ok = n1 >= la && n1 <= l_last && (n1 < own_a || n1 > own_b);
                measure(box1, ok ? n1 : l_last);
                m1 = __ballot(ok && near() == (sweep == 1) && reaches());
                if (wait > 0) {
                    --wait;
                } else if (m1) {
                    uint64_t which = m1 & kProbe ? m1 & kProbe : m1;
                    for (bool probe = true;; probe = false) {
                        const int32_t tested = __popcll(which);
                        m1 = each_query(m1, which);
                        if (!probe) break;
                        const bool pays = 3 * (tested - __popcll(m1 & which)) >= tested;
                        pause = pays ? 0 : min(2 * pause + 1, 63);
                        which = m1 & ~which;
                        if (!pays || !which) break;
                    }
                    wait = pause;
                }
            } else if (m3) {
                first2 = (first3 + __builtin_ctzll(m3)) << 6;
                m3 &= m3 - 1;
                const int32_t n2 = first2 + lane;
                bool ok = n2 >= (la >> 6) && n2 <= (l_last >> 6);
                if (tree.has2) {
                    measure(box2, ok ? n2 : (l_last >> 6));
                    ok = ok && (sweep > 1 || near()) && reaches();
                }
                m2 = __ballot(ok);
                if (tree.has2) m2 = each_query(m2, m2);
            } else if (t3 <= (l_last >> 12)) {
                first3 = t3;
                const int32_t n3 = t3 + lane;
                t3 += 64;
                bool ok = n3 <= (l_last >> 12);
                if (tree.has3) {
                    measure(box3, ok ? n3 : (l_last >> 12));
                    ok = ok && (sweep > 1 || near()) && reaches();
                }
                m3 = __ballot(ok);
            } else {
                return false;
            }
        }
        return true;
    };
    Raw ahead;
    bool have = false;
    for (;;) {
        const bool run = have;
        const int32_t leaf0 = ahead.leaf0, leaf1 = ahead.leaf1;
        Frag a0, a1;
        float a_scale = scale;
        auto convert = [&](const Raw& r) __attribute__((always_inline)) {
            float w[NV * 4];
#pragma unroll
            for (int v = 0; v < NV; ++v) { w[4 * v] = r.v[v].x; w[4 * v + 1] = r.v[v].y; w[4 * v + 2] = r.v[v].z; w[4 * v + 3] = r.v[v].w; }
            bool live = r.live;
            if (a.dir) live = live && dir_is_neighbour(a.dir[__float_as_int(w[D])]);
            float c[D];
#pragma unroll
            for (int i = 0; i < D; ++i) c[i] = fminf(fmaxf(__builtin_fmaf(w[i], scale, -zs[i]), -32.0f), 32.0f);
            float h = half_norm<D>(c);
            h = live ? h : (float)kLeafBigH;
            const float hh = half_lo(pack_half(h, 0.0f));
            uint32_t s[8];
            pack_slots<D>(c, hh, h - hh, 1.0f, 1.0f, s);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a0.u[i] = s[i];
                a1.u[i] = s[i + 4];
                swap_halves(a0.u[i], a1.u[i]);
            }
            a_scale = scale;
        };
        if (run) convert(ahead);
        have = advance();
        if (have) {          // the next two leaves are requested before these are compared (two pairs ahead: no gain)
            const int32_t l0 = first1 + __builtin_ctzll(m1);
            m1 &= m1 - 1;
            const int32_t l1 = m1 ? first1 + __builtin_ctzll(m1) : -1;
            m1 &= m1 - 1;
            ahead = fetch(l0, l1);
        }
        if (run) {
#pragma unroll 1
            for (int blk = 0;; ++blk) {
                const int32_t leaf = blk ? leaf1 : leaf0;
                const bool last = blk == 1 || leaf1 < 0;
                Frag A;
#pragma unroll
                for (int i = 0; i < 4; ++i) A.u[i] = blk ? a1.u[i] : a0.u[i];
                const acc16_t zero = {};
                const acc16_t f0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A.h, b0.h, zero, 0, 0, 0);
                const acc16_t f1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A.h, b1.h, zero, 0, 0, 0);
                uint32_t s0 = signs(f0), s1 = signs(f1);
                swap_halves(s0, s1);
                uint32_t m = s0 | (s1 << 16);
                const int32_t base = leaf * kLeafPts;
                // Only the query's own row split: where the tile spans several, and at either end (there the filter has
                // refused what lies outside already; this keeps a position beyond the last point out of the queue by itself)
                if (several || base < pa || base + kLeafPts > pb) {
                    const int32_t from = max(ends[lane] - base, 0), to = min(ends[kQueryBlock + lane] - base, 32);
                    const uint64_t range = to > from ? ((1ull << to) - 1) & ~((1ull << from) - 1) : 0ull;
                    m &= (uint32_t)range;
                }
                --excess;
                if (__builtin_expect(exact, 0)) m = sift(base, m);
                while (m) {
                    queue[cnt * kQueryBlock + lane] = (uint32_t)(base + __builtin_ctz(m));
                    m &= m - 1;
                    ++cnt;
                }
                // at the end of a sweep everything queued is merged
                const int32_t trig = last && !have ? 1 : kLeafTrig;
                if (__any(cnt >= trig)) {
                    do {
                        absorb();
                        ++excess;
                    } while (__any(cnt >= trig));
                    exact = exact || excess > kLeafSiftFrom || (excess > kLeafSiftTies && !__any(active && tau_hi != 0));
                    m1 &= __ballot(reaches());
                }
                if (last) break;
                if (scale != a_scale) {                  // a merge has changed the scale: the second block once more
                    convert(fetch(leaf0, leaf1));
                }
            }
        }
        if (!have) {                                     // sweep over
            if (++sweep == 3) break;
            if (sweep == 1) {
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    near_limit[g] = uniform_value<(KC > 48)>(gtau[g] < 0 ? -1.0f : (gtau[g] < 0x7f800000 ? __int_as_float(gtau[g]) * 0.015625f : hext * hext));
            }
            t3 = la >> 12;
        }
    }
    }   // any query searches

    write_tile_rows<KC>(a, best, lds64, my_row, valid, asks, cap, few, 0u);
}

// EITHER: the call may be the group kernel's.  An instantiation of its own: the test in front moved the loops of every call, 500k
// points, d = 8, K = 64 9672 -> 9829 us, 60k, d = 10, K = 40 1249 -> 1273 (and without it again as before).
template <int D, int KC, bool LOWER, bool EITHER>
__global__ void __launch_bounds__(kQueryBlock) __attribute__((amdgpu_waves_per_eu(leaf_waves<KC>(), leaf_waves<KC>())))
k_query_leaf(QueryArgs a, LeafTree tree)
{
    extern __shared__ uint64_t lds64[];
    if constexpr (EITHER) {
        if (leaf_not_asked<D>(a)) {
            if (a.dir && threadIdx.x == 0) a.handed[blockIdx.x] = 0;
            return;
        }
    }
    const bool dense = D == 2 && a.dense_class > 0;      // only the heaviest tiles, in the order of the ranking kernels
    const int32_t count = dense ? dense_tiles(a) : 0;
    int32_t i = blockIdx.x;
    if (dense && i >= count) return;
    do {
        int32_t tile = i;
        if (dense) {
            tile = a.tile_order[i] & ((1 << kOrderFlagBit) - 1);
        } else if (tile < (int32_t)(gridDim.x & ~127u)) {
            // Neighbouring tiles read the same leaves: runs of 16 tiles go to one XCD (workgroups are dealt round robin to 8)
            // so that they meet in its L2 (runs of 4 to 256: the same within 3 %; heaviest tiles first, as the tile
            // kernel takes them: 500k uniform points, d = 8, K = 64 17.4 against 15.3 ms).
            const int32_t xcd = tile & 7, j = tile >> 3;
            tile = ((j >> 4) * 8 + xcd) * 16 + (j & 15);
        }
        leaf_tile<D, KC, LOWER>(a, tree, tile, lds64);
        if (!dense) break;
        __syncthreads();
        i += gridDim.x;
    } while (i < count);
}

// With direction flags: tiles of which no more queries than this ask hand them to the list kernel.  A tile costs nearly the same
// however few of its queries ask; the list kernel costs so much a query, which grows with the points around it from d = 8
// on.  One uniform split, a tile's cost over a query's: d = 6, 50k to 1M points 30 to 38; d = 8, 50k 35 to 41, 200k 16
// (K = 64) and 20 (K = 16), 1M 6 to 9; d = 10, 50k 20 to 28.  One in ten asking: 200k points, d = 6, K = 64 2.05 -> 0.42 ms
// (tile kernel 1.15); 1M, d = 6, K = 16 8.3 -> 1.5 (2.5); 50k, d = 10, K = 40 1.15 -> 0.62 (2.0).  Half of them asking, d = 6,
// the tile kernel would be the faster one (1M, K = 16 5.4 against 7.6 ms; d = 8 45 against 17), but the share is
// known on the device only.
static inline int32_t leaf_few_ask(int32_t d, int32_t n, int32_t n_segments, int32_t k_list)
{
    const int32_t split = n / n_segments;
    if (d <= 7) return 32;
    return split <= 1 << 16 ? 24 : (split <= 1 << 18 ? (k_list > 32 ? 12 : 16) : 6);
}

template <int D, bool LOWER>
static hipError_t launch_leaf_pass(const QueryArgs& a_in, hipStream_t stream)
{
    QueryArgs a = a_in;
    const LeafTree t = leaf_tree(a.work_list, a.n);
    int grid = (a.n + kQueryBlock - 1) / kQueryBlock;
    if (a.dense_class > 0 && grid > kDenseGrid) grid = kDenseGrid;      // its workgroups take further tiles
    if (!LOWER || a.dense_class > 0 || a.dir) {       // the second pass of a long list finds the boxes of the first, unless the work list took their place
        constexpr int NB = box_vecs<D>();
        const int box_grid = (a.n + 255) / 256;
        FG_LAUNCH(k_leaf_boxes<D>, dim3(a.dense_class > 0 && box_grid > kDenseGrid ? kDenseGrid : box_grid), dim3(256), 0, stream, a, t.boxes);
        float4* const box2 = t.boxes + (int64_t)t.n1 * NB;
        if (t.has2) FG_LAUNCH(k_node_boxes<D>, dim3((t.n2 + 3) / 4), dim3(256), 0, stream, a, t.boxes, t.n1, box2, t.n2);
        if (t.has3) FG_LAUNCH(k_node_boxes<D>, dim3((t.n3 + 3) / 4), dim3(256), 0, stream, a, box2, t.n2, box2 + (int64_t)t.n2 * NB, t.n3);
    }
    const int32_t cap = a.k_list;
    a.few_ask = leaf_few_ask(D, a.n, a.n_segments, a.k_list);
#define FG_LEAF(KC, EITHER) FG_LAUNCH((k_query_leaf<D, KC, LOWER, EITHER>), dim3(grid), dim3(kQueryBlock), (leaf_lds_bytes<KC, D>()), stream, a, t)
#define FG_LEAF_LISTS(EITHER)         \
    if (cap <= 16) FG_LEAF(16, EITHER);      \
    else if (cap <= 32) FG_LEAF(32, EITHER); \
    else if (cap <= 48) FG_LEAF(48, EITHER); \
    else FG_LEAF(64, EITHER)
    if constexpr (D > kClustersMaxD) {
        if (a.votes) {
            FG_LEAF_LISTS(true);
            return hipSuccess;
        }
    }
    FG_LEAF_LISTS(false);
#undef FG_LEAF_LISTS
#undef FG_LEAF
    return hipSuccess;
}

}  // namespace fg
