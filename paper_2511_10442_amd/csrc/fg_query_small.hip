// Small problems: one wavefront per query, every point of its row split a candidate.  No bins, no boxes, one launch.
//
// At a thousand points the tile kernel is one wavefront per tile on a sixteenth of the CUs, 37 us from its first shell to
// its last row, behind six binning launches of 3 to 9 us each; comparing every pair is a few microseconds of the whole
// chip.  The list is the one of the list kernel: one key per lane, ascending.  256 candidates are requested at a time
// (four per lane), so a thousand points are four trips to memory.
// REC: candidates are the bin-ordered records of a binning, else the caller's coordinates in their own order.
#include "fg_query_list.hpp"

namespace fg {

constexpr int kSmallBatch = 4;

template <int D, bool REC>
__global__ void __launch_bounds__(kQueryBlock)
k_query_small(QueryArgs a)
{
    const int lane = threadIdx.x;
    const int32_t p = blockIdx.x;
    if (REC && p == 0 && lane == 0) *a.work_count = 0;              // nothing is handed over
    const int32_t seg = segment_of(a.row_splits, a.n_segments, p);
    const int32_t sa = a.row_splits[seg], sb = a.row_splits[seg + 1];
    auto load = [&](int32_t q, float (&y)[D], int32_t& row) __attribute__((always_inline)) {
        if constexpr (REC) load_rec<D>(a.rec, q, y, row);
        else {
#pragma unroll
            for (int c = 0; c < D; ++c) y[c] = a.coords[(int64_t)q * D + c];
            row = q;
        }
    };
    float x[D];
    int32_t row;
    load(p, x, row);
    const int32_t cap = a.k_list;                                   // 0 <= cap <= 64
    const bool asks = !(a.dir && !dir_is_query(a.dir[row]));
    uint64_t best = lane >= kQueryBlock - cap ? kEmptyKey : 0ull;   // ascending by lane, low lanes pinned
    uint64_t tau = wave_last_key(best);
    // batches in cyclic order from the query's own: in bin order the near ones come first and fewer keys enter the list
    constexpr int32_t kStep = kSmallBatch * kQueryBlock;
    const int32_t batches = asks ? (sb - sa + kStep - 1) / kStep : 0;
    int32_t base = sa + (p - sa) / kStep * kStep;
    for (int32_t i = 0; i < batches; ++i, base = base + kStep < sb ? base + kStep : sa) {
        float y[kSmallBatch][D];
        int32_t src[kSmallBatch];
        bool live[kSmallBatch];
#pragma unroll
        for (int u = 0; u < kSmallBatch; ++u) {
            const int32_t q = base + u * kQueryBlock + lane;
            live[u] = q < sb && q != p;
            load(live[u] ? q : p, y[u], src[u]);
        }
        if (a.dir) {
#pragma unroll
            for (int u = 0; u < kSmallBatch; ++u) live[u] = live[u] && dir_is_neighbour(a.dir[src[u]]);
        }
#pragma unroll
        for (int u = 0; u < kSmallBatch; ++u) {
            float diff = x[0] - y[u][0];
            float d2 = diff * diff;
#pragma unroll
            for (int c = 1; c < D; ++c) {
                diff = x[c] - y[u][c];
                d2 = d2 + diff * diff;
            }
            const uint64_t key = ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)src[u];
            const bool acc = live[u] && key < tau;
            uint64_t m = __ballot(acc);
            if (m == 0) continue;
            if (__popcll(m) <= kListDirect) {       // few: one at a time, as in the list kernel
                do {
                    const int b = __ffsll((unsigned long long)m) - 1;
                    m &= m - 1;
                    const uint64_t in = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(key >> 32), b) << 32) |
                                        (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, b);
                    best = key_min(best, key_max(in, wave_from_below(best)));
                } while (m);
            } else {
                const uint64_t v = wave_sort64(acc ? key : kEmptyKey, lane);
                best = wave_merge64(key_min(__shfl(v, kQueryBlock - 1 - lane, 64), best), lane);
            }
            tau = wave_last_key(best);
        }
    }
    int32_t* oi = a.out_idx + (int64_t)row * a.k;
    float* od = a.out_d2 + (int64_t)row * a.k;
    if (lane == 0) { oi[0] = asks ? row : -1; od[0] = 0.0f; }
    if (lane >= kQueryBlock - cap) {
        const int32_t j = lane - (kQueryBlock - cap) + 1;
        const bool real = best < kEmptyKey;
        oi[j] = real ? (int32_t)(uint32_t)best : -1;
        od[j] = real ? __uint_as_float((uint32_t)(best >> 32)) : 0.0f;
    }
}

template <int D>
static hipError_t launch_small(const QueryArgs& a, hipStream_t stream)
{
    if (a.coords) FG_LAUNCH((k_query_small<D, false>), dim3(a.n), dim3(kQueryBlock), 0, stream, a);
    else FG_LAUNCH((k_query_small<D, true>), dim3(a.n), dim3(kQueryBlock), 0, stream, a);
    return hipSuccess;
}

hipError_t launch_query_small(const QueryArgs& a_in, hipStream_t stream)
{
    QueryArgs a = a_in;
    a.slot0 = 0;
    a.k_list = a.k - 1;
    switch (a.d) {
        case 2: return launch_small<2>(a, stream);
        case 3: return launch_small<3>(a, stream);
        case 4: return launch_small<4>(a, stream);
        case 5: return launch_small<5>(a, stream);
        case 6: return launch_small<6>(a, stream);
        case 7: return launch_small<7>(a, stream);
        case 8: return launch_small<8>(a, stream);
        case 9: return launch_small<9>(a, stream);
        case 10: return launch_small<10>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fg
