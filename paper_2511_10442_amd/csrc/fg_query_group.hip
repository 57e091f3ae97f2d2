// Group kernel: one wavefront for two or four consecutive bin-ordered queries, candidates one per lane.
//
// Same result as the other query kernels (paper Section 3, Algorithm 2: the exact K-1 best others by (distance, index)).
// For the sizes at which one wavefront for 64 queries (tile and leaf kernel) leaves the chip short of wavefronts, or of which
// few dense tiles set the end: 20,000 points are 313 tiles on 1024 SIMDs, and 10,000 groups here.
//   * The sorted points are cut into leaves of 64 consecutive points, one per lane, with bounding boxes over all d
//     coordinates, and 64 leaves form a node (k_group_boxes).  Everything about a query is wave-uniform: its coordinates sit
//     in scalar registers, its list is one key per lane, ascending, and candidates are compared 64 at a time.
//   * The bound that decides what is kept comes before the first candidate is kept: of the 64 leaves around the queries' own
//     the eight nearest are looked at for every lane's nearest candidate, and the cap-th smallest of these 64 distances (one
//     sort of a word per lane) has cap candidates at or below it.  Lists that fill from empty kept twice as many.
//   * Then the leaves that still reach: those eight, the ones within half the bound's distance, the rest.  Kept candidates
//     wait in LDS until 64 are there (or the sweep ends) and are sorted and merged across the lanes (fg_wavesort.hpp).
// What bounds it: vector issue, 69 % of the SIMDs' slots at 20,000 uniform points, d = 3, K = 32, and 94 % at 100,000 (1130 and 1330
// instructions a query by the counters; as the code has it a third the sorts of 230 each, a third distances, 14 for 64 candidates,
// the rest box tests and bounds); below, the chain of one group.  A bound from a first pass over the near leaves as well (nothing kept until
// then, then one sort a query) cost more distances than it saved sorts: +10 to +80 %.  Figures beside the rule,
// takes_group_kernel.
#include "fg_query_tile.hpp"
#include "fg_group_boxes.hpp"
#include "fg_wavesort.hpp"

namespace fg {

// Leaves that a first bound comes from.  Query stage for 4 / 8 / 16, in us: uniform points, d = 3, 20k, K = 32 108 / 69 / 69, 100k 277 / 257 / 315; d = 4, 40k, K = 40
// 206 / 184 / 192; d = 6, 40k, K = 20 366 / 358 / 359; 100k points in showers, K = 32 341 / 228 / 265, in a mixture, d = 4, K = 40 475 / 381 / 402.
constexpr int kGroupStart = 8;
// Most workgroups where there may be nothing to do: an empty launch of 8192, 16384 and 25,000 takes 3, 5 and 7 us, and clusters of 100k
// points, d = 4, K = 40 455, 395 and 385 (each takes further groups, whose number differs by one).
constexpr int32_t kRankedGrid = 16384;
constexpr int kGroupPend = 128;                 // kept candidates of a query between two merges

// EITHER: unless the leaf kernel has served the call (an instantiation of its own: 0.4 us of every call's 10)
template <int D, bool EITHER>
static __global__ void __launch_bounds__(1024)
k_group_boxes(const float4* __restrict__ rec, int32_t n, GroupTree tree, int32_t* __restrict__ work_count, const int32_t* votes, int32_t votes_for)
{
    if (EITHER && *votes < votes_for) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) *work_count = 0;         // nothing is handed over on this path
    group_boxes<D, 16>(rec, n, tree, blockIdx.x);
}

__device__ __forceinline__ int32_t uniform_i32(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// a wave-uniform value kept in a vector register: the scalar ones are what this kernel is short of
__device__ __forceinline__ float in_vector(float v) { asm("" : "+v"(v)); return v; }

template <int D, int Q, bool LOWER, bool CHOICE>
__device__ __forceinline__ void group_queries(const QueryArgs& a, const GroupTree& tree, const int32_t p0, uint64_t (*pend)[kGroupPend])
{
    constexpr int NV = rec_vecs(D);
    constexpr int NB = group_box_vecs<D>();
    const int lane = threadIdx.x;
    const int32_t cap = a.k_list;                   // 0 <= cap <= 64
    const float kInf = __int_as_float(0x7f800000);
    // lane q of the first Q holds query q
    float x[D];
    int32_t row;
    load_rec<D>(a.rec, min(p0 + min(lane, Q - 1), a.n - 1), x, row);
    const bool asks = p0 + lane < a.n && lane < Q && !(a.dir && !dir_is_query(a.dir[row]));
    const uint32_t asking = cap > 0 ? (uint32_t)__ballot(asks) : 0u;              // bit q
    uint64_t best[Q], lower[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) { best[q] = kEmptyKey; lower[q] = 0; }
    if (LOWER) {
        uint64_t l = 0;
        if (asks) {
            const int32_t li = a.out_idx[(int64_t)row * a.k + a.slot0];
            l = li < 0 ? kEmptyKey : (((uint64_t)__float_as_uint(a.out_d2[(int64_t)row * a.k + a.slot0]) << 32) | (uint32_t)li);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            lower[q] = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(l >> 32), q) << 32) | (uint32_t)__builtin_amdgcn_readlane((int32_t)l, q);
    }
    float xs[Q][D];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int c = 0; c < D; ++c) xs[q][c] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[c]), q));

    int32_t seg, sb;
    {   // row split of the first query: 64 of the boundaries at a time
        int32_t lo = 0, hi = a.n_segments;
        while (hi - lo > 1) {
            const int32_t step = (hi - lo + 63) >> 6;
            const int32_t at = lo + (lane + 1) * step;
            const int32_t c = __popcll(__ballot(at < hi && a.row_splits[at] <= p0));
            lo += c * step;
            hi = min(hi, lo + step);
        }
        seg = lo;
        sb = uniform_i32(a.row_splits[lo]);
    }
    // the queries of one row split at a time (nearly always all of them)
    uint32_t todo = asking;
    while (todo) {
    const int32_t first_q = p0 + __builtin_ctz(todo);
    int32_t sa = sb;
    do {                                            // (the split of the first query left, and empty ones passed over)
        sa = uniform_i32(a.row_splits[seg]);
        sb = uniform_i32(a.row_splits[++seg]);
    } while (first_q >= sb);
    const uint32_t act = sb - p0 >= Q ? todo : todo & ((1u << (sb - p0)) - 1);
    todo &= ~act;

    const int32_t la = sa / kGroupLeaf, lb = (sb - 1) / kGroupLeaf;               // leaves of the split, inclusive
    const int32_t own = p0 / kGroupLeaf;
    float tau[Q], near[Q];                          // a candidate farther than tau cannot enter the list; -1: not searching
    uint32_t tie[Q];                                // one at tau can up to this index
    int32_t np[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        tau[q] = in_vector((act >> q) & 1 ? kInf : -1.0f);
        near[q] = in_vector(0.0f);
        tie[q] = 0xffffffffu;
        np[q] = 0;
    }
    // which lanes of a leaf hold candidates of query q
    auto live_lanes = [&](int q, int32_t base) __attribute__((always_inline)) -> uint64_t {
        uint64_t m = ~0ull;
        if (base < sa || base + kGroupLeaf > sb || base == own * kGroupLeaf) {
            const int32_t from = max(sa - base, 0), to = min(sb - base, 64);
            m = to >= 64 ? ~0ull : (1ull << to) - 1;
            m &= ~0ull << from;
            const int32_t self = p0 + q - base;
            if (base == own * kGroupLeaf) m &= ~(1ull << self);
        }
        return m;
    };
    auto distance = [&](int q, const float (&w)[NV * 4]) __attribute__((always_inline)) -> float {
        float diff = xs[q][0] - w[0];
        float d2 = diff * diff;
#pragma unroll
        for (int c = 1; c < D; ++c) {
            diff = xs[q][c] - w[c];
            d2 = d2 + diff * diff;
        }
        return d2;
    };
    auto load_leaf = [&](int32_t leaf, float (&w)[NV * 4]) __attribute__((always_inline)) {
        const int64_t at = min(leaf * kGroupLeaf + lane, a.n - 1);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const float4 f = a.rec[at * NV + v];
            w[4 * v] = f.x; w[4 * v + 1] = f.y; w[4 * v + 2] = f.z; w[4 * v + 3] = f.w;
        }
    };
    // the lane's number, afresh: else every comparison of it in the sorts below is kept in scalar registers throughout
    auto here = [&]() __attribute__((always_inline)) -> int { int l = threadIdx.x; asm volatile("" : "+v"(l)); return l; };
    // merges the oldest 64 kept candidates of a query into its list
    auto absorb = [&](int q) __attribute__((always_inline)) {
        const int lane = here();
        __syncthreads();
        const uint64_t v = lane < np[q] ? pend[q][lane] : kEmptyKey;
        const uint64_t rest = lane + 64 < np[q] ? pend[q][lane + 64] : 0ull;
        __syncthreads();
        if (lane + 64 < np[q]) pend[q][lane] = rest;
        np[q] = max(np[q] - 64, 0);
        best[q] = wave_merge_lists(best[q], wave_sort64_dpp(v, lane), lane);
        const uint32_t kth = (uint32_t)__builtin_amdgcn_readlane((int32_t)(best[q] >> 32), cap - 1);
        if (kth <= (uint32_t)uniform_i32(__float_as_int(tau[q]))) {      // (above it while the list is open or has a gap)
            tau[q] = in_vector(__uint_as_float(kth));
            tie[q] = (uint32_t)__builtin_amdgcn_readlane((int32_t)best[q], cap - 1);
        }
    };
    float b2[Q];
    auto measure = [&](const float4* __restrict__ boxes, int32_t i) __attribute__((always_inline)) {
        float w[NB * 4];
#pragma unroll
        for (int v = 0; v < NB; ++v) {
            const float4 f = boxes[(int64_t)i * NB + v];
            w[4 * v] = f.x; w[4 * v + 1] = f.y; w[4 * v + 2] = f.z; w[4 * v + 3] = f.w;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float s = 0.0f;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const float gap = fmaxf(fmaxf(w[c] - xs[q][c], xs[q][c] - w[D + c]), 0.0f);
                s = c == 0 ? gap * gap : __builtin_fmaf(gap, gap, s);
            }
            b2[q] = s;
        }
    };
    // The leaves to start with: of the 64 around the queries' own those whose boxes are nearest to one of the queries.
    const int32_t win = max(min(own - 32, lb - 63), la);
    uint64_t start;
    {
        const int lane = here();
        const bool ok = win + lane <= lb;
        measure(tree.leaf, ok ? win + lane : lb);
        float d = 3.0e38f;
#pragma unroll
        for (int q = 0; q < Q; ++q) d = (act >> q) & 1 ? fminf(d, b2[q]) : d;
        const uint32_t key = ok ? (__float_as_uint(d) & ~63u) | (uint32_t)lane : 0x7fffffffu;
        const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int32_t)wave_sort64_words(key, lane), kGroupStart - 1);
        start = __ballot(ok && key <= last);
    }
    // A first bound: every lane's nearest of these leaves; the cap-th smallest of these 64 distances has cap candidates at or
    // below it.
    {
        uint32_t low[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) low[q] = 0x7f800000u;
        for (uint64_t m = start; m; m &= m - 1) {
            const int32_t leaf = win + __builtin_ctzll(m);
            float w[NV * 4];
            load_leaf(leaf, w);
            const uint64_t can = a.dir ? __ballot(dir_is_neighbour(a.dir[__float_as_int(w[D])])) : ~0ull;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (!((act >> q) & 1)) continue;
                const uint32_t bits = __float_as_uint(distance(q, w));
                const uint64_t m = live_lanes(q, leaf * kGroupLeaf) & can;
                bool in = (m >> lane) & 1;
                if (LOWER) in = in && (((uint64_t)bits << 32) | __float_as_uint(w[D])) > lower[q];
                if (in) low[q] = min(low[q], bits);
            }
        }
        const int lane = here();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if ((act >> q) & 1) tau[q] = in_vector(__int_as_float(__builtin_amdgcn_readlane((int32_t)wave_sort64_words(low[q], lane), cap - 1)));
        }
    }

    // sweep 0: the leaves to start with; 1: leaves whose box is near; 2: the others that a list still reaches
    int32_t sweep = 0, first = win;
    uint64_t mask[Q], all = start;
#pragma unroll
    for (int q = 0; q < Q; ++q) mask[q] = (act >> q) & 1 ? all : 0ull;
    const int32_t na = la >> 6, nb = lb >> 6;       // nodes, inclusive
    int32_t node64 = nb + 1;                        // next 64 nodes to test (in sweep 0: none)
    uint64_t nodes = 0;
    // Boxes whose points cannot enter the list of query q are farther than this: the k-th best, enlarged for the rounding of
    // distances and bounds (2^-17 where 2^-18 are needed); squares below 1e-30 have lost their relative accuracy.
    auto reach = [&](int q) __attribute__((always_inline)) -> float { return fmaxf(tau[q] * 1.0000077f, 1e-30f); };
    // the next 64 leaves with something in them; false: the sweep is over
    auto advance = [&]() __attribute__((always_inline)) -> bool {
        while (!all) {
            if (nodes) {
                const int32_t node = node64 - 64 + __builtin_ctzll(nodes);
                nodes &= nodes - 1;
                first = node << 6;
                const int32_t l = first + lane;
                const uint32_t i = (uint32_t)(l - win);
                const bool ok = l >= la && l <= lb && (i > 63 || !((start >> i) & 1));
                const uint64_t in = __ballot(ok);
                measure(tree.leaf, ok ? l : lb);
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const uint64_t nr = __ballot(b2[q] <= near[q]);
                    mask[q] = sweep == 1 ? nr : __ballot(b2[q] <= reach(q)) & ~nr;
                    mask[q] = (act >> q) & 1 ? mask[q] & in : 0ull;
                    all |= mask[q];
                }
            } else if (node64 <= nb) {
                const int32_t i = node64 + lane;
                node64 += 64;
                nodes = __ballot(i <= nb);
                if (nb - na > 1 && ((CHOICE && D > kClustersMaxD) || !a.votes)) {   // (with the tiles' votes the nodes have no boxes)
                    measure(tree.node, min(i, nb));
                    uint64_t hit = 0;
#pragma unroll
                    for (int q = 0; q < Q; ++q)
                        if ((act >> q) & 1) hit |= __ballot(b2[q] <= (sweep == 1 ? near[q] : reach(q)));
                    nodes &= hit;
                }
            } else {
                return false;
            }
        }
        return true;
    };
    float w[NV * 4];
    int32_t leaf;
    uint32_t who;                                   // queries that want it
    auto pop = [&](int32_t& l, uint32_t& wh) __attribute__((always_inline)) {
        const int b = __builtin_ctzll(all);
        all &= all - 1;
        l = first + b;
        wh = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) wh |= (uint32_t)((mask[q] >> b) & 1) << q;
    };
    pop(leaf, who);
    load_leaf(leaf, w);
    for (;;) {
        // the next leaf is requested before this one is looked at
        float wn[NV * 4];
        int32_t next = -1;
        uint32_t who_next = 0;
        if (advance()) {
            pop(next, who_next);
            load_leaf(next, wn);
        }
        const int32_t base = leaf * kGroupLeaf;
        const uint64_t can = a.dir ? __ballot(dir_is_neighbour(a.dir[__float_as_int(w[D])])) : ~0ull;
        {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (!((who >> q) & 1)) continue;
                const float d2 = distance(q, w);
                uint64_t m = __ballot(d2 <= tau[q]) & live_lanes(q, base) & can;
                if (m) {
                    const uint64_t key = ((uint64_t)__float_as_uint(d2) << 32) | __float_as_uint(w[D]);
                    bool in = __longlong_as_double((long long)key) <= __longlong_as_double((long long)(((uint64_t)__float_as_uint(tau[q]) << 32) | tie[q]));
                    if (LOWER) in = in && key > lower[q];
                    m &= __ballot(in);
                    const int32_t at = np[q] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                    if ((m >> lane) & 1) pend[q][at] = key;
                    np[q] += __popcll(m);
                }
            }
            const int32_t limit = next >= 0 ? 64 : (sweep == 0 ? 24 : 0);
            bool more;
            do {
                more = false;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (np[q] > limit) { absorb(q); more = more || np[q] > limit; }
                }
            } while (more);
        }
        if (next < 0) {
            if (sweep == 2) break;
            do {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (sweep == 0) near[q] = in_vector(tau[q] * 0.25f);         // (an open list: everything is near)
                ++sweep;
                node64 = na;
                nodes = 0;
            } while (!advance() && sweep < 2);
            if (!all) break;
            pop(next, who_next);
            load_leaf(next, wn);
        }
        leaf = next;
        who = who_next;
#pragma unroll
        for (int c = 0; c < NV * 4; ++c) w[c] = wn[c];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) while (np[q] > 0) absorb(q);
    }   // queries of one row split

    if (lane < Q && p0 + lane < a.n && a.slot0 == 0) {
        a.out_idx[(int64_t)row * a.k] = asks || (cap == 0 && !(a.dir && !dir_is_query(a.dir[row]))) ? row : -1;
        a.out_d2[(int64_t)row * a.k] = 0.0f;
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (p0 + q >= a.n) break;
        const int64_t at = (int64_t)__builtin_amdgcn_readlane(row, q) * a.k + a.slot0 + 1 + lane;
        if (lane < cap) {
            const bool real = best[q] < kEmptyKey;
            a.out_idx[at] = real ? (int32_t)(uint32_t)best[q] : -1;
            a.out_d2[at] = real ? __uint_as_float((uint32_t)(best[q] >> 32)) : 0.0f;
        }
    }
}

// With a.dense_class (d >= 6: votes) only if the tiles are this kernel's, all or none; ranked tiles in their order, of which the workgroups take groups in turn,
// and those of a tile meet in one XCD's L2 (workgroups are dealt round robin to 8).
// CHOICE: the device decides whether it does anything (from six dimensions on an instantiation of its own, as its tests move the loops of every call:
// 24k points in a mixture, d = 6, K = 50 309 -> 313 us).
template <int D, int Q, bool LOWER, bool CHOICE>
__global__ void __launch_bounds__(kQueryBlock)
k_query_group(QueryArgs a, GroupTree tree)
{
    constexpr int kPerTile = kQueryBlock / Q;
    __shared__ uint64_t pend[Q][kGroupPend];
    const bool asked = CHOICE && (D > kClustersMaxD || a.dense_class > 0), ranked = asked && !a.votes;
    const int32_t count = asked ? dense_tiles(a) : 0;
    if (asked && count == 0) return;
    const int32_t rounds = ranked ? (count + 7) >> 3 : 0;
    const int32_t groups = ranked ? rounds * 8 * kPerTile : (int32_t)gridDim.x;
    // heaviest tiles first, and whoever has the first of one round has the last of the next
    for (int32_t round = 0; round * (int32_t)gridDim.x < groups; ++round) {
        const int32_t i = round * gridDim.x + (round & 1 ? gridDim.x - 1 - blockIdx.x : blockIdx.x);
        int32_t p0 = i * Q;
        if (ranked) {
            const int32_t j = i >> 3, at = (j / kPerTile) * 8 + (i & 7);
            p0 = at < count ? (a.tile_order[at] & ((1 << kOrderFlagBit) - 1)) * kQueryBlock + (j % kPerTile) * Q : a.n;
        }
        if (p0 < a.n) group_queries<D, Q, LOWER, CHOICE>(a, tree, p0, pend);
        if (!ranked) break;
        __syncthreads();
    }
}

template <int D, int Q>
static hipError_t launch_group_pass(const QueryArgs& a, const GroupTree& tree, hipStream_t stream)
{
    int32_t blocks = (a.n + Q - 1) / Q;
    if (a.dense_class > 0 && blocks > kRankedGrid) blocks = kRankedGrid;       // its workgroups take further groups
    const dim3 grid(blocks);
    constexpr bool either = D <= kClustersMaxD;      // one instantiation for both
    if (either || a.votes) {
        if (a.slot0 == 0) FG_LAUNCH((k_query_group<D, Q, false, true>), grid, dim3(kQueryBlock), 0, stream, a, tree);
        else FG_LAUNCH((k_query_group<D, Q, true, true>), grid, dim3(kQueryBlock), 0, stream, a, tree);
    } else {
        if (a.slot0 == 0) FG_LAUNCH((k_query_group<D, Q, false, either>), grid, dim3(kQueryBlock), 0, stream, a, tree);
        else FG_LAUNCH((k_query_group<D, Q, true, either>), grid, dim3(kQueryBlock), 0, stream, a, tree);
    }
    return hipSuccess;
}

// Two queries a wavefront where four would leave the chip short of wavefronts, and from seven dimensions on, where the second
// pair's state costs more (102 vector registers at d = 10) than the shared loads and box tests save.  Query stage, four against
// two, in us: 10k points, K = 40: d = 3 49 against 40, d = 5 (20k) 142 / 142; 40k, d = 3 111 / 116, d = 5 267 / 268, d = 8 831 / 722.
constexpr int32_t kGroupPairsN = 16384;

// Direction flags, six dimensions and more: a.votes and, where half of the points ask or few are anyone's neighbours, as many more as make
// the call the group kernel's.  (One workgroup, some 5 us for 60,000 flags.)  Few neighbours lie far apart, and the leaf kernel hands
// its queries to the list kernel, which goes through the empty bins between them.  Whole call, leaf and list against group kernel, uniform points of which
// the same share asks and is neighbour, in us: d = 6, K = 24, 22k, 1 % 995 / 304, 10 % 476 / 270, 40k, 1 % 947 / 508, 10 % 313 / 426; d = 8, K = 40, 40k, 1 %
// 617 / 471, 10 % 521 / 700.
constexpr int32_t kFewNeighbours = 2500;

static __global__ void __launch_bounds__(1024) k_ask_votes(QueryArgs a, const int32_t* __restrict__ votes, int32_t* __restrict__ out)
{
    __shared__ int32_t total[2];
    if (threadIdx.x < 2) total[threadIdx.x] = 0;
    __syncthreads();
    int32_t ask = 0, answer = 0;
#pragma unroll 4
    for (int32_t i = threadIdx.x; i < a.n; i += 1024) {
        const int32_t flag = a.dir[i];
        ask += dir_is_query(flag) ? 1 : 0;
        answer += dir_is_neighbour(flag) ? 1 : 0;
    }
    ask = wave_sum_i32(ask);
    answer = wave_sum_i32(answer);
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&total[0], ask);
        atomicAdd(&total[1], answer);
    }
    __syncthreads();
    if (threadIdx.x == 0) *out = *votes + (2 * total[0] >= a.n || total[1] < kFewNeighbours ? a.n : 0);
}

hipError_t launch_ask_votes(const QueryArgs& a, const int32_t* votes, int32_t* out, hipStream_t stream)
{
    FG_LAUNCH(k_ask_votes, dim3(1), dim3(1024), 0, stream, a, votes, out);
    return hipSuccess;
}

template <int D>
static hipError_t launch_group(const QueryArgs& a_in, hipStream_t stream)
{
    QueryArgs a = a_in;
    const GroupTree tree = group_tree<D>(a.work_list, a.n);
    if (D > kClustersMaxD && a.votes) FG_LAUNCH((k_group_boxes<D, (D > kClustersMaxD)>), dim3(tree.n_node), dim3(1024), 0, stream, a.rec, a.n, tree, a.work_count, a.votes, a.votes_for);
    else FG_LAUNCH((k_group_boxes<D, false>), dim3(tree.n_node), dim3(1024), 0, stream, a.rec, a.n, tree, a.work_count, nullptr, 0);
    const int32_t cap = a.k - 1;
    for (a.slot0 = 0; a.slot0 == 0 || a.slot0 < cap; a.slot0 += 64) {
        a.k_list = cap - a.slot0 < 64 ? cap - a.slot0 : 64;
        if (D >= 7 || a.n <= kGroupPairsN) FG_TRY((launch_group_pass<D, 2>(a, tree, stream)));
        else if constexpr (D < 7) FG_TRY((launch_group_pass<D, 4>(a, tree, stream)));
    }
    return hipSuccess;
}

template <int D>
static hipError_t launch_clusters(const QueryArgs& a, hipStream_t stream)
{
    return launch_group_pass<D, 4>(a, group_tree<D>(a.work_list, a.n), stream);
}

hipError_t launch_query_clusters(const QueryArgs& a, hipStream_t stream)
{
    switch (a.d) {
        case 2: return launch_clusters<2>(a, stream);
        case 3: return launch_clusters<3>(a, stream);
        case 4: return launch_clusters<4>(a, stream);
        case 5: return launch_clusters<5>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_query_group(const QueryArgs& a, hipStream_t stream)
{
    switch (a.d) {
        case 2: return launch_group<2>(a, stream);
        case 3: return launch_group<3>(a, stream);
        case 4: return launch_group<4>(a, stream);
        case 5: return launch_group<5>(a, stream);
        case 6: return launch_group<6>(a, stream);
        case 7: return launch_group<7>(a, stream);
        case 8: return launch_group<8>(a, stream);
        case 9: return launch_group<9>(a, stream);
        case 10: return launch_group<10>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fg
