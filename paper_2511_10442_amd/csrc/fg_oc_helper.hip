// Object-condensation index matrices (paper Section 5, Algorithm 3).
//
// For every object candidate k the vertices of its row split are walked from `tid` vertices
// into the window, wrapping round; members go to row k of M, non-members to row k of M_not,
// both padded with -1.  Entry `fill` of row k is stored at fill * n_unique + k (the paper's
// index macro), so neighbouring objects are neighbouring addresses.
//
// The paper runs one thread per object over its whole row split: with a few thousand objects
// that is a few dozen wavefronts, each a chain of 1e5 dependent steps.  Here the walk is cut
// into chunks so that (objects / 64) x (chunks) wavefronts run at once:
//   count    members of object k inside walk chunk c                    -> counts[c][k]
//   scan     exclusive prefix over the chunks of every object           -> members before chunk c, total
//   members  walk chunk c again and write the members at their final row of M; pad M with -1
//   others   for a block of OUTPUT rows of M_not: row r of an object holds the vertex at walk position r + m(r),
//            m(r) = members met before the r-th non-member, a step function that M itself tells (member j at walk
//            position w_j comes before row r iff w_j - j <= r).  So nothing is walked, but for objects with more members
//            than M has rows: the steps of 32 rows go through LDS and the rows are written with a running sum.
// Lanes are objects throughout, so objects of one row split read neighbouring vertices; all objects of a wavefront that
// share a window read it through scalar loads (count, members).
// Integer-only; bound by the M_not write stream (n_unique x n_maxrs words).  10 x 100,000 vertices, 2,000 objects,
// 0.82 GB: 800 -> 395 us (count 100 -> 34, scan 56 -> 11, members 171 -> 49, others 509 -> 294, of which the stores
// alone would take some 160).
// Without a workspace the single-kernel form of the paper is used.
#include "fg_internal.hpp"

namespace fg {

constexpr int kOcBlock = 64;
constexpr int kOcBatch = 8;       // independent loads kept in flight per lane
constexpr int kOcChunk = 128;     // walk positions per chunk

struct OcWindow { int32_t uq, start, len, rot; };

__device__ __forceinline__ OcWindow oc_window(int32_t k, const int32_t* __restrict__ unique_idx,
                                              const int32_t* __restrict__ unique_rs_asso, const int32_t* __restrict__ rs,
                                              int32_t n_vert, int32_t n_splits, int32_t n_maxrs, int32_t rot_block)
{
    OcWindow w;
    w.uq = unique_idx[k];
    int32_t split = unique_rs_asso[k];
    split = split < 0 ? 0 : (split >= n_splits ? n_splits - 1 : split);    // out-of-range split: clamped, never read outside rs
    int32_t start = rs[split], end = rs[split + 1];
    start = start < 0 ? 0 : start;
    if (end > n_vert) end = n_vert;
    if (end - start > n_maxrs) end = start + n_maxrs;
    w.start = start;
    w.len = end > start ? end - start : 0;
    const int32_t tid = k % rot_block;
    w.rot = tid < w.len ? tid : 0;          // a start past the window means the window in order
    return w;
}

// vertex at walk position p (0 <= p < len)
__device__ __forceinline__ int32_t oc_vertex(const OcWindow& w, int32_t p)
{
    int32_t o = w.rot + p;
    if (o >= w.len) o -= w.len;
    return w.start + o;
}

// ---- single kernel, one lane per object (no workspace) ---------------------------------------
__global__ void __launch_bounds__(kOcBlock)
k_oc_helper(const int32_t* __restrict__ asso_idx, const int32_t* __restrict__ unique_idx,
            const int32_t* __restrict__ unique_rs_asso, const int32_t* __restrict__ rs, int32_t n_vert,
            int32_t n_unique, int32_t n_splits, int32_t n_maxuq, int32_t n_maxrs, int32_t calc_m_not,
            int32_t rot_block, int32_t* __restrict__ M, int32_t* __restrict__ M_not)
{
    const int32_t k = blockIdx.x * kOcBlock + threadIdx.x;
    if (k >= n_unique) return;
    const OcWindow w = oc_window(k, unique_idx, unique_rs_asso, rs, n_vert, n_splits, n_maxrs, rot_block);
    int32_t fill = 0, fill_not = 0;
    for (int32_t p = 0; p < w.len; ++p) {
        const int32_t i = oc_vertex(w, p);
        if (asso_idx[i] == w.uq) {
            if (fill < n_maxuq) { M[(int64_t)fill * n_unique + k] = i; ++fill; }
        } else if (calc_m_not) {
            M_not[(int64_t)fill_not * n_unique + k] = i;      // fill_not < len <= n_maxrs
            ++fill_not;
        }
    }
    for (; fill < n_maxuq; ++fill) M[(int64_t)fill * n_unique + k] = -1;
    if (calc_m_not)
        for (; fill_not < n_maxrs; ++fill_not) M_not[(int64_t)fill_not * n_unique + k] = -1;
}

// ---- chunked form ----------------------------------------------------------------------------
// The walk of a chunk is the same for all objects with the same window and no rotation, and a wavefront's 64 objects
// have few windows unless row splits hold only a handful of objects each.  Then every window is walked once with scalar
// loads (a vector compare and a conditional add a position instead of an address, a gather and a compare per lane).
constexpr int kOcFewWindows = 4;
__device__ __forceinline__ bool oc_few_windows(const OcWindow& w)
{
    if (__any(w.rot != 0)) return false;
    bool todo = true;
    for (int i = 0; i < kOcFewWindows; ++i) {
        if (todo) {
            const int32_t start = __builtin_amdgcn_readfirstlane(w.start), len = __builtin_amdgcn_readfirstlane(w.len);
            if (w.start == start && w.len == len) todo = false;
        }
        if (!__any(todo)) return true;
    }
    return false;
}
// f(walk position, vertex label) for every position of the chunk that starts at p0, in order
template <typename F>
__device__ __forceinline__ void oc_each_window(const OcWindow& w, int32_t p0, F f, const int32_t* __restrict__ asso_idx)
{
    bool todo = true;
    while (todo) {
        const int32_t start = __builtin_amdgcn_readfirstlane(w.start), len = __builtin_amdgcn_readfirstlane(w.len);
        if (w.start != start || w.len != len) continue;
        todo = false;
        const int32_t p1 = p0 + kOcChunk < len ? p0 + kOcChunk : len;
        const int32_t* const at = asso_idx + start;
        int32_t p = p0;
        for (; p + kOcBatch <= p1; p += kOcBatch) {
            int32_t v[kOcBatch];
#pragma unroll
            for (int u = 0; u < kOcBatch; ++u) v[u] = at[p + u];
#pragma unroll
            for (int u = 0; u < kOcBatch; ++u) f(p + u, v[u]);
        }
        for (; p < p1; ++p) f(p, at[p]);
    }
}

// grid (object groups, chunks); counts[c][k] = members of k at walk positions [c*C, (c+1)*C)
__global__ void __launch_bounds__(kOcBlock)
k_oc_count(const int32_t* __restrict__ asso_idx, const int32_t* __restrict__ unique_idx,
           const int32_t* __restrict__ unique_rs_asso, const int32_t* __restrict__ rs, int32_t n_vert, int32_t n_unique,
           int32_t n_splits, int32_t n_maxrs, int32_t rot_block, int32_t* __restrict__ counts)
{
    const int32_t k = blockIdx.x * kOcBlock + threadIdx.x;
    if (k >= n_unique) return;
    const OcWindow w = oc_window(k, unique_idx, unique_rs_asso, rs, n_vert, n_splits, n_maxrs, rot_block);
    const int32_t p0 = blockIdx.y * kOcChunk;
    const int32_t p1 = p0 + kOcChunk < w.len ? p0 + kOcChunk : w.len;
    int32_t c = 0;
    if (oc_few_windows(w)) {
        oc_each_window(w, p0, [&](int32_t, int32_t v) { c += v == w.uq; }, asso_idx);
    } else {
        for (int32_t pb = p0; pb < p1; pb += kOcBatch) {       // loads of a batch are independent: all in flight at once
            int32_t v[kOcBatch];
#pragma unroll
            for (int u = 0; u < kOcBatch; ++u) v[u] = pb + u < p1 ? asso_idx[oc_vertex(w, pb + u)] : ~w.uq;
#pragma unroll
            for (int u = 0; u < kOcBatch; ++u) c += v[u] == w.uq;
        }
    }
    counts[(int64_t)blockIdx.y * n_unique + k] = c;
}

// One block per 64 objects, a lane each: counts[c][k] -> members before chunk c; counts[n_chunks][k] = all members.  The 16
// wavefronts take a sixteenth of the chunks each: sums, then prefixes from the sums of the wavefronts before (one
// wavefront alone is a chain of a hundred trips to memory at 100,000 vertices: 56 -> 11 us).
constexpr int kOcScanWaves = 16;
__global__ void __launch_bounds__(kOcBlock * kOcScanWaves)
k_oc_scan(int32_t* __restrict__ counts, int32_t n_unique, int32_t n_chunks)
{
    __shared__ int32_t sums[kOcScanWaves][kOcBlock];
    const int lane = threadIdx.x & (kOcBlock - 1), wv = threadIdx.x / kOcBlock;
    const int32_t k = blockIdx.x * kOcBlock + lane;
    const int32_t part = (n_chunks + kOcScanWaves - 1) / kOcScanWaves;
    const int32_t c0 = wv * part, c1 = c0 + part < n_chunks ? c0 + part : n_chunks;
    int32_t sum = 0;
    if (k < n_unique) {
#pragma unroll 8
        for (int32_t c = c0; c < c1; ++c) sum += counts[(int64_t)c * n_unique + k];
    }
    sums[wv][lane] = sum;
    __syncthreads();
    if (k >= n_unique) return;
    int32_t run = 0, total = 0;
    for (int j = 0; j < kOcScanWaves; ++j) {
        if (j < wv) run += sums[j][lane];
        total += sums[j][lane];
    }
    for (int32_t cb = c0; cb < c1; cb += kOcBatch) {
        int32_t t[kOcBatch];
#pragma unroll
        for (int u = 0; u < kOcBatch; ++u) t[u] = cb + u < c1 ? counts[(int64_t)(cb + u) * n_unique + k] : 0;
#pragma unroll
        for (int u = 0; u < kOcBatch; ++u) {
            if (cb + u < c1) counts[(int64_t)(cb + u) * n_unique + k] = run;
            run += t[u];
        }
    }
    if (wv == 0) counts[(int64_t)n_chunks * n_unique + k] = total;
}

// grid (object groups, chunks + pad blocks): chunk blocks write the members of their chunk at their final rows; a pad
// block fills its kOcPadRows rows of M with -1 past each object's last member (all rows in one block per object group
// was a chain of thousands of stores and 150 of the kernel's 171 us)
constexpr int kOcPadRows = 64;
__global__ void __launch_bounds__(kOcBlock)
k_oc_members(const int32_t* __restrict__ asso_idx, const int32_t* __restrict__ unique_idx,
             const int32_t* __restrict__ unique_rs_asso, const int32_t* __restrict__ rs, int32_t n_vert, int32_t n_unique,
             int32_t n_splits, int32_t n_maxuq, int32_t n_maxrs, int32_t rot_block, int32_t n_chunks,
             const int32_t* __restrict__ counts, int32_t* __restrict__ M)
{
    const int32_t k = blockIdx.x * kOcBlock + threadIdx.x;
    if (k >= n_unique) return;
    if ((int32_t)blockIdx.y >= n_chunks) {
        const int32_t total = counts[(int64_t)n_chunks * n_unique + k];
        for (int64_t r0 = ((int64_t)blockIdx.y - n_chunks) * kOcPadRows; r0 < n_maxuq; r0 += (int64_t)(gridDim.y - n_chunks) * kOcPadRows) {
            const int32_t r1 = r0 + kOcPadRows < n_maxuq ? (int32_t)r0 + kOcPadRows : n_maxuq;
            for (int32_t r = (int32_t)r0 > total ? (int32_t)r0 : total; r < r1; ++r) M[(int64_t)r * n_unique + k] = -1;
        }
        return;
    }
    const OcWindow w = oc_window(k, unique_idx, unique_rs_asso, rs, n_vert, n_splits, n_maxrs, rot_block);
    const int32_t p0 = blockIdx.y * kOcChunk;
    const int32_t p1 = p0 + kOcChunk < w.len ? p0 + kOcChunk : w.len;
    int32_t fill = counts[(int64_t)blockIdx.y * n_unique + k];
    if (oc_few_windows(w)) {
        oc_each_window(w, p0, [&](int32_t p, int32_t v) {
            if (v == w.uq && fill < n_maxuq) { M[(int64_t)fill * n_unique + k] = w.start + p; ++fill; }
        }, asso_idx);
        return;
    }
    for (int32_t pb = p0; pb < p1 && fill < n_maxuq; pb += kOcBatch) {
        int32_t v[kOcBatch];
#pragma unroll
        for (int u = 0; u < kOcBatch; ++u) v[u] = pb + u < p1 ? asso_idx[oc_vertex(w, pb + u)] : ~w.uq;
#pragma unroll
        for (int u = 0; u < kOcBatch; ++u)
            if (v[u] == w.uq && fill < n_maxuq) { M[(int64_t)fill * n_unique + k] = oc_vertex(w, pb + u); ++fill; }
    }
}

// One wavefront per 64 objects and `rows` output rows of M_not, a lane each, kOcTile rows at a time: first every lane
// adds its object's steps to its column of an LDS table (steps[i] = members that come before row i and after row i - 1),
// then the rows are written with a running sum.  A step is a member of the list in M, or, for an object with more members
// than M has rows, a member met on a walk over the vertices; each lane goes at its own pace through its own steps, and
// however unevenly members are spread, all objects write the same row at the same time.  The first steps of the next rows
// are requested before the present rows are written.
// (Steps in registers, refilled by the whole wavefront whenever one of its objects had used four: 302 us at 10 x 100,000
// vertices and 2,000 objects, but 16 times the walk's time with few objects, whose members lie close.)
constexpr int kOcTile = 32;
constexpr int kOcAhead = 4;
constexpr int kOcOthersWaves = 4096;
__global__ void __launch_bounds__(kOcBlock)
k_oc_others(const int32_t* __restrict__ asso_idx, const int32_t* __restrict__ unique_idx,
            const int32_t* __restrict__ unique_rs_asso, const int32_t* __restrict__ rs, int32_t n_vert, int32_t n_unique,
            int32_t n_splits, int32_t n_maxuq, int32_t n_maxrs, int32_t rot_block, int32_t n_chunks, int32_t rows,
            const int32_t* __restrict__ counts, const int32_t* __restrict__ M, int32_t* __restrict__ M_not)
{
    __shared__ int32_t steps[kOcTile][kOcBlock];
    const int lane = threadIdx.x;
    const int32_t k = blockIdx.x * kOcBlock + lane;
    if (k >= n_unique) return;
    const int32_t r0 = blockIdx.y * rows;
    const int32_t r1 = r0 + rows < n_maxrs ? r0 + rows : n_maxrs;
    const OcWindow w = oc_window(k, unique_idx, unique_rs_asso, rs, n_vert, n_splits, n_maxrs, rot_block);
    const int32_t total = counts[(int64_t)n_chunks * n_unique + k];
    const bool listed = total <= n_maxuq;          // M holds every member
    // the row before which member q comes: its walk position less the members before it
    auto row_of = [&](int32_t vertex, int32_t q) -> int32_t {
        int32_t o = vertex - w.start - w.rot;
        if (o < 0) o += w.len;
        return o - q;
    };
    auto entry = [&](int32_t q) -> int32_t { return M[(int64_t)q * n_unique + k]; };
    // q: members before row r0
    int32_t q = 0;
    if (listed) {
        for (int32_t hi = total; q < hi;) {        // rows of the members ascend: halving
            const int32_t mid = (q + hi) >> 1;
            if (row_of(entry(mid), mid) < r0) q = mid + 1; else hi = mid;
        }
    } else {
        // the last chunk with at most r0 non-members before it, then on to the place right after non-member r0 - 1
        int32_t lo = 0, hi = n_chunks;
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (mid * kOcChunk - counts[(int64_t)mid * n_unique + k] <= r0) lo = mid; else hi = mid;
        }
        int32_t p = lo * kOcChunk;
        q = counts[(int64_t)lo * n_unique + k];
        while (p < w.len && p - q < r0) {
            int32_t v[kOcBatch];
#pragma unroll
            for (int u = 0; u < kOcBatch; ++u) v[u] = p + u < w.len ? asso_idx[oc_vertex(w, p + u)] : w.uq;
#pragma unroll
            for (int u = 0; u < kOcBatch; ++u) {
                if (p < w.len && p - q < r0) { q += v[u] == w.uq; ++p; }
            }
        }
    }
    int32_t next[kOcAhead];
    auto request = [&]() {
#pragma unroll
        for (int u = 0; u < kOcAhead; ++u) next[u] = listed && q + u < total ? entry(q + u) : 0;
    };
    request();
#pragma unroll
    for (int i = 0; i < kOcTile; ++i) steps[i][lane] = 0;
    int32_t before = q;
    for (int32_t rb = r0; rb < r1; rb += kOcTile) {
        const int32_t re = rb + kOcTile;
        // false: the step (if there is one) belongs to a later row
        auto step_at = [&](int32_t row) -> bool {
            if (row >= re) return false;
            atomicAdd(&steps[row - rb][lane], 1);      // the lane's own word: only so that nothing waits for a result
            ++q;
            return true;
        };
        if (listed) {
            bool open = true;
#pragma unroll
            for (int u = 0; u < kOcAhead; ++u) open = open && q < total && step_at(row_of(next[u], q));
            while (open) {
                int32_t v[kOcBatch];
#pragma unroll
                for (int u = 0; u < kOcBatch; ++u) v[u] = q + u < total ? entry(q + u) : 0;
#pragma unroll
                for (int u = 0; u < kOcBatch; ++u) open = open && q < total && step_at(row_of(v[u], q));
            }
            request();
        } else {
            int32_t p = rb + q;
            while (p < w.len && p - q < re) {
                int32_t v[kOcBatch];
#pragma unroll
                for (int u = 0; u < kOcBatch; ++u) v[u] = p + u < w.len ? asso_idx[oc_vertex(w, p + u)] : w.uq;
#pragma unroll
                for (int u = 0; u < kOcBatch; ++u) {
                    if (p < w.len && p - q < re) {
                        if (v[u] == w.uq) step_at(p - q);
                        ++p;
                    }
                }
            }
        }
        int32_t* at = M_not + (int64_t)rb * n_unique + k;
        const int32_t some = re < r1 ? kOcTile : r1 - rb;
        for (int32_t i0 = 0; i0 < some; i0 += kOcBatch) {
            int32_t s[kOcBatch];
#pragma unroll
            for (int u = 0; u < kOcBatch; ++u) { s[u] = steps[i0 + u][lane]; steps[i0 + u][lane] = 0; }
#pragma unroll
            for (int u = 0; u < kOcBatch; ++u) {
                before += s[u];
                const int32_t p = rb + i0 + u + before;
                if (i0 + u < some) *at = p < w.len ? oc_vertex(w, p) : -1;
                at += n_unique;
            }
        }
    }
}

size_t oc_workspace_bytes(int64_t n_unique, int32_t n_maxrs)
{
    const int64_t n_chunks = (n_maxrs + kOcChunk - 1) / kOcChunk;
    return (size_t)(n_chunks + 1) * (size_t)n_unique * sizeof(int32_t);
}

hipError_t launch_oc_helper(const int32_t* asso_idx, const int32_t* unique_idx, const int32_t* unique_rs_asso,
                            const int32_t* rs, int32_t n_vert, int32_t n_unique, int32_t n_splits, int32_t n_maxuq,
                            int32_t n_maxrs, int32_t calc_m_not, int32_t rot_block, int32_t* M, int32_t* M_not,
                            int32_t* counts, hipStream_t stream)
{
    const unsigned groups = (unsigned)((n_unique + kOcBlock - 1) / kOcBlock);
    const int32_t n_chunks = (n_maxrs + kOcChunk - 1) / kOcChunk;
    if (!counts || n_chunks + 1 > 65535) {
        FG_LAUNCH(k_oc_helper, dim3(groups), dim3(kOcBlock), 0, stream, asso_idx, unique_idx, unique_rs_asso, rs,
                  n_vert, n_unique, n_splits, n_maxuq, n_maxrs, calc_m_not, rot_block, M, M_not);
        return hipSuccess;
    }
    FG_LAUNCH(k_oc_count, dim3(groups, n_chunks), dim3(kOcBlock), 0, stream, asso_idx, unique_idx, unique_rs_asso,
              rs, n_vert, n_unique, n_splits, n_maxrs, rot_block, counts);
    FG_LAUNCH(k_oc_scan, dim3(groups), dim3(kOcBlock * kOcScanWaves), 0, stream, counts, n_unique, n_chunks);
    int64_t pads = ((int64_t)n_maxuq + kOcPadRows - 1) / kOcPadRows;
    if (pads > 65535 - n_chunks) pads = 65535 - n_chunks;
    FG_LAUNCH(k_oc_members, dim3(groups, n_chunks + (unsigned)pads), dim3(kOcBlock), 0, stream, asso_idx, unique_idx,
              unique_rs_asso, rs, n_vert, n_unique, n_splits, n_maxuq, n_maxrs, rot_block, n_chunks, counts, M);
    if (calc_m_not) {
        // rows per wavefront: its search for the first one is paid once, but the chip holds some 5000 of these wavefronts
        int32_t rows = 4 * kOcTile;
        while (rows > kOcTile && (int64_t)groups * ((n_maxrs + rows - 1) / rows) < kOcOthersWaves) rows >>= 1;
        FG_LAUNCH(k_oc_others, dim3(groups, (unsigned)((n_maxrs + (int64_t)rows - 1) / rows)), dim3(kOcBlock), 0, stream,
                  asso_idx, unique_idx, unique_rs_asso, rs, n_vert, n_unique, n_splits, n_maxuq, n_maxrs, rot_block,
                  n_chunks, rows, counts, M, M_not);
    }
    return hipSuccess;
}

}  // namespace fg
