// Order inside dense cells: a cell's points may stand in any order, and where a cell holds many they are put along a
// space-filling curve, so that runs of consecutive points have small bounding boxes.
//
// The leaf kernel rules out runs of 32 points by their boxes.  Bins are made for some K points at the mean density; where the
// density varies by orders of magnitude a bin holds 10^4 to 10^5 points, and in the order of their arrival every run of
// those has the whole bin's box: 5M points of density r^(-5/3), d = 2, K = 16 compared up to 10^5 candidates a query.
//   k_order_split   cells of more than kOrderChunk points, a workgroup each: bounding box, 2^12 sub-cells of it in Morton order
//                   (counted in LDS, rows scattered), and the same for every sub-cell of more than kOrderChunk points.  The
//                   box is that of the points, so a step resolves a density that no regular grid does.
//   k_order_chunk   cells and runs of sub-cells of up to kOrderChunk points: sorted in LDS by their place along the curve,
//                   records written.
// The lists of cells come from the prefix sum (k_scan_apply).  Without dense cells the two launches find empty lists: some 5 us.
// What bounds it: the fullest cell, whose first steps one workgroup takes alone (184 us where a split of a million has 5 10^4
// points in a cell; a far outlier that puts nearly all points of a split into one cell leaves the ordering to one CU, at some
// 3.7 ns a point), then the sorts (136 us for 1.3 10^6 points).  5M such points, d = 2, K = 16: fg_bin_points 680 -> 970 us, query
// 10,750 -> 2700, backward (whose rows follow the order) 1130 -> 613.
#include "fg_internal.hpp"
#include "fg_order.hpp"

namespace fg {

constexpr int kSplitThreads = 1024;
constexpr int kSplitWaves = kSplitThreads / 64;
constexpr int kSplitBits = 12;                    // sub-cells of a step: 2^12 counters in LDS
constexpr int kSplitCodes = 1 << kSplitBits;
constexpr int kSplitLevels = 8;                   // steps at most: bounds the list of chunks
constexpr int kOrderWindow = kOrderChunk / 2;     // sub-cells of up to so many points share a chunk with those that start in the same window
constexpr int kChunkThreads = 256;
constexpr int kChunkItems = kOrderChunk / kChunkThreads;
constexpr int kSplitGrid = 256;
constexpr int kChunkGrid = 4096;

// place of a quantised point along the curve: bits of the coordinates interleaved, highest first
template <int D, int BITS>
__device__ __forceinline__ uint32_t curve_place(const uint32_t (&q)[D])
{
    uint32_t f = 0;
#pragma unroll
    for (int b = BITS - 1; b >= 0; --b)
#pragma unroll
        for (int c = 0; c < D; ++c) f = (f << 1) | ((q[c] >> b) & 1u);
    return f;
}

template <int D, int BITS>
__device__ __forceinline__ uint32_t place_in_box(const float (&x)[D], const float (&lo)[D], const float (&scale)[D])
{
    uint32_t q[D];
#pragma unroll
    for (int c = 0; c < D; ++c) q[c] = (uint32_t)fminf(fmaxf((x[c] - lo[c]) * scale[c], 0.0f), (float)((1u << BITS) - 1));   // (NaN: 0)
    return curve_place<D, BITS>(q);
}
// cells per unit length, 0 where the points do not differ; `sides` the number of cells
__device__ __forceinline__ float place_scale(float lo, float hi, float sides)
{
    const float ext = hi - lo;
    return ext > 0.0f && ext <= 3.0e38f ? fminf(sides / ext, 3.0e38f) : 0.0f;
}

__device__ __forceinline__ float order_wave_min(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}

// minima and maxima over a workgroup of W wavefronts, in all threads
template <int D, int W>
__device__ __forceinline__ void block_box(float (&mn)[D], float (&mx)[D], float (*red)[2 * D])
{
    const int wv = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < D; ++c) {
        const float a = order_wave_min(mn[c]), b = order_wave_min(-mx[c]);
        if ((threadIdx.x & 63) == 0) { red[wv][c] = a; red[wv][D + c] = b; }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < D; ++c) {
        float a = red[0][c], b = red[0][D + c];
#pragma unroll
        for (int w = 1; w < W; ++w) { a = fminf(a, red[w][c]); b = fminf(b, red[w][D + c]); }
        mn[c] = a;
        mx[c] = -b;
    }
}

// row and coordinates of the point at position p of a piece: from its record, or from a list of rows
template <int D>
__device__ __forceinline__ int32_t order_point(const float4* __restrict__ rec, const int32_t* rows, const float* __restrict__ coords, int32_t p, float (&x)[D])
{
    int32_t row;
    if (!rows) {
        load_rec<D>(rec, p, x, row);
    } else {
        row = rows[p];
#pragma unroll
        for (int c = 0; c < D; ++c) x[c] = coords[(int64_t)row * D + c];
    }
    return row;
}

__device__ __forceinline__ uint32_t order_wave_scan(uint32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}
// sum of the threads below, the total in *total
__device__ __forceinline__ uint32_t split_scan(uint32_t v, uint32_t* wave_tot, uint32_t* total)
{
    const int wv = threadIdx.x >> 6;
    const uint32_t inc = order_wave_scan(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 63) wave_tot[wv] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
        const uint32_t t = wave_tot[w];
        if (w < wv) base += t;
        tot += t;
    }
    *total = tot;
    return base + inc - v;
}
// maximum of the threads below, 0 in the first
__device__ __forceinline__ uint32_t split_max_below(uint32_t v, uint32_t* wave_tot)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t m = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(m, o, 64);
        if (lane >= o) m = max(m, t);
    }
    uint32_t below = __shfl_up(m, 1, 64);
    below = lane == 0 ? 0u : below;
    __syncthreads();
    if (lane == 63) wave_tot[wv] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w)
        if (w < wv) below = max(below, wave_tot[w]);
    return below;
}

template <int D>
static __global__ void __launch_bounds__(kSplitThreads)
k_order_split(OrderArgs a)
{
    constexpr int BITS = kSplitBits / D;
    constexpr int CODES = 1 << (BITS * D);
    constexpr int PER = (CODES + kSplitThreads - 1) / kSplitThreads;
    __shared__ uint32_t count[kSplitCodes];       // population of a sub-cell, then where its next point goes
    __shared__ uint32_t edge[kSplitCodes + 1];    // first positions of chunks and (lowest bit set) of larger sub-cells, doubled
    __shared__ float red[kSplitWaves][2 * D];
    __shared__ uint32_t wave_tot[kSplitWaves];
    __shared__ int32_t stacked;
    const int t = threadIdx.x;
    const int32_t n_large = a.counters[kOrderLarge];
    for (int32_t task = blockIdx.x; task < n_large; task += gridDim.x) {
        const int32_t cell = a.large[task];
        const int32_t first = a.bounds[cell], end = a.bounds[cell + 1];
        // Pieces still to be split, three words each.  They are disjoint and of more than kOrderChunk points: 3 L / 2049 <= L / 256 - 2
        // words for a cell of L > 2048.
        int32_t* const stack = a.stack + (first + 255) / 256;
        __syncthreads();
        if (t == 0) { stack[0] = first; stack[1] = end - first; stack[2] = 0; stacked = 1; }
        __syncthreads();
        for (;;) {
            const int32_t top = stacked;
            if (top == 0) break;
            const int32_t p0 = stack[3 * top - 3], len = stack[3 * top - 2], level = stack[3 * top - 1];
            const int32_t* const src = level == 0 ? nullptr : ((level & 1) ? a.rows0 : a.rows1);
            int32_t* const dst = (level & 1) ? a.rows1 : a.rows0;
            __syncthreads();
            if (t == 0) stacked = top - 1;
            for (int i = t; i < CODES; i += kSplitThreads) count[i] = 0;
            float lo[D], hi[D], scale[D];
#pragma unroll
            for (int c = 0; c < D; ++c) { lo[c] = 3.4028235e38f; hi[c] = -3.4028235e38f; }
#pragma unroll 4
            for (int32_t i = t; i < len; i += kSplitThreads) {
                float x[D];
                order_point<D>(a.rec, src, a.coords, p0 + i, x);
#pragma unroll
                for (int c = 0; c < D; ++c) { lo[c] = fminf(lo[c], x[c]); hi[c] = fmaxf(hi[c], x[c]); }
            }
            block_box<D, kSplitWaves>(lo, hi, red);
#pragma unroll
            for (int c = 0; c < D; ++c) scale[c] = place_scale(lo[c], hi[c], (float)(1 << BITS));
#pragma unroll 4
            for (int32_t i = t; i < len; i += kSplitThreads) {
                float x[D];
                order_point<D>(a.rec, src, a.coords, p0 + i, x);
                atomicAdd(&count[place_in_box<D, BITS>(x, lo, scale)], 1u);
            }
            __syncthreads();
            uint32_t num[PER], at[PER], sum = 0, total;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const int code = t * PER + j;
                num[j] = code < CODES ? count[code] : 0u;
                sum += num[j];
            }
            uint32_t run = split_scan(sum, wave_tot, &total);
            uint32_t last = 0;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                at[j] = run;
                const int code = t * PER + j;
                if (code < CODES) count[code] = run;
                run += num[j];
                if (num[j]) last = (at[j] << 1 | (num[j] > kOrderWindow ? 1u : 0u)) + 1u;
            }
            // A chunk is a run of sub-cells of up to kOrderWindow points that start in the same window of kOrderWindow positions, so it
            // has less than kOrderChunk; a larger sub-cell stands by itself (and is longer than what is left of the window).
            uint32_t before = split_max_below(last, wave_tot);
            uint32_t opens[PER], n_open = 0;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const bool large = num[j] > kOrderWindow;
                const bool head = num[j] && (large || before == 0 || ((before - 1) & 1) || (before - 1) >> 1 >> kOrderWindowShift != at[j] >> kOrderWindowShift);
                opens[j] = head ? 1u : 0u;
                n_open += opens[j];
                if (num[j]) before = (at[j] << 1 | (large ? 1u : 0u)) + 1u;
            }
            uint32_t n_edges;
            uint32_t slot = split_scan(n_open, wave_tot, &n_edges);
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (opens[j]) edge[slot++] = at[j] << 1 | (num[j] > kOrderWindow ? 1u : 0u);
            if (t == 0) edge[n_edges] = (uint32_t)len << 1;
            __syncthreads();
            for (uint32_t e = t; e < n_edges; e += kSplitThreads) {
                const int32_t from = (int32_t)(edge[e] >> 1), m = (int32_t)(edge[e + 1] >> 1) - from;
                if (m > kOrderChunk && m < len && level + 1 < kSplitLevels) {
                    const int32_t s = atomicAdd(&stacked, 1);
                    stack[3 * s] = p0 + from; stack[3 * s + 1] = m; stack[3 * s + 2] = level + 1;
                } else if (m < len || level > 0) {
                    // (more than kOrderChunk only of points that are not told apart: by equal coordinates, or after the last step)
                    const int32_t parts = (m + kOrderChunk - 1) / kOrderChunk;
                    const int32_t to = atomicAdd(&a.counters[kOrderChunks], parts);
                    for (int32_t i = 0; i < parts; ++i)
                        a.chunks[to + i] = make_int4(p0 + from + i * kOrderChunk, min(kOrderChunk, m - i * kOrderChunk), 1 + (level & 1), 0);
                }
            }
#pragma unroll 4
            for (int32_t i = t; i < len; i += kSplitThreads) {
                float x[D];
                const int32_t row = order_point<D>(a.rec, src, a.coords, p0 + i, x);
                dst[p0 + (int32_t)atomicAdd(&count[place_in_box<D, BITS>(x, lo, scale)], 1u)] = row;
            }
            __syncthreads();
        }
    }
}

template <int D>
static __global__ void __launch_bounds__(kChunkThreads)
k_order_chunk(OrderArgs a)
{
    constexpr int BITS = 32 / D;
    constexpr int NV = rec_vecs(D);
    __shared__ uint64_t key[kOrderChunk];
    __shared__ float red[kChunkThreads / 64][2 * D];
    const int t = threadIdx.x;
    const int32_t n_small = a.counters[kOrderSmall], n_tasks = n_small + a.counters[kOrderChunks];
    for (int32_t task = blockIdx.x; task < n_tasks; task += gridDim.x) {
        int32_t first, len, from = 0;
        if (task < n_small) {
            const int32_t cell = a.small[task];
            first = a.bounds[cell];
            len = a.bounds[cell + 1] - first;
        } else {
            const int4 c = a.chunks[task - n_small];
            first = c.x; len = c.y; from = c.z;
        }
        const int32_t* const src = from == 0 ? nullptr : (from == 1 ? a.rows0 : a.rows1);
        float x[kChunkItems][D];
        int32_t row[kChunkItems];
        float lo[D], hi[D], scale[D];
#pragma unroll
        for (int c = 0; c < D; ++c) { lo[c] = 3.4028235e38f; hi[c] = -3.4028235e38f; }
#pragma unroll
        for (int j = 0; j < kChunkItems; ++j) {
            const int32_t i = j * kChunkThreads + t;
            row[j] = order_point<D>(a.rec, src, a.coords, first + min(i, len - 1), x[j]);
        }
#pragma unroll
        for (int j = 0; j < kChunkItems; ++j)
#pragma unroll
            for (int c = 0; c < D; ++c) { lo[c] = fminf(lo[c], x[j][c]); hi[c] = fmaxf(hi[c], x[j][c]); }
        block_box<D, kChunkThreads / 64>(lo, hi, red);
#pragma unroll
        for (int c = 0; c < D; ++c) scale[c] = place_scale(lo[c], hi[c], (float)(1u << BITS));
        int32_t size = kChunkThreads;                                  // what is sorted: a power of two
        while (size < len) size <<= 1;
#pragma unroll
        for (int j = 0; j < kChunkItems; ++j) {
            const int32_t i = j * kChunkThreads + t;
            if (i < size) key[i] = i < len ? ((uint64_t)place_in_box<D, BITS>(x[j], lo, scale) << 32) | (uint32_t)row[j] : ~0ull;
        }
        __syncthreads();
        for (int32_t block = 2; block <= size; block <<= 1) {
            for (int32_t half = block >> 1; half > 0; half >>= 1) {
                for (int32_t p = t; p < size >> 1; p += kChunkThreads) {
                    const int32_t i = 2 * p - (p & (half - 1));
                    const uint64_t u = key[i], v = key[i + half];
                    if ((u > v) == ((i & block) == 0)) { key[i] = v; key[i + half] = u; }
                }
                __syncthreads();
            }
        }
        for (int32_t i = t; i < len; i += kChunkThreads) {
            const int32_t r = (int32_t)(uint32_t)key[i];
            float w[NV * 4];
#pragma unroll
            for (int c = 0; c < NV * 4; ++c) w[c] = 0.0f;
#pragma unroll
            for (int c = 0; c < D; ++c) w[c] = a.coords[(int64_t)r * D + c];
            w[D] = __int_as_float(r);
#pragma unroll
            for (int v = 0; v < NV; ++v) a.rec[(int64_t)(first + i) * NV + v] = make_float4(w[4 * v], w[4 * v + 1], w[4 * v + 2], w[4 * v + 3]);
        }
        __syncthreads();
    }
}

hipError_t launch_order(const OrderArgs& a, hipStream_t stream)
{
    FG_LAUNCH(k_order_split<2>, dim3(kSplitGrid), dim3(kSplitThreads), 0, stream, a);
    FG_LAUNCH(k_order_chunk<2>, dim3(kChunkGrid), dim3(kChunkThreads), 0, stream, a);
    return hipSuccess;
}

}  // namespace fg
