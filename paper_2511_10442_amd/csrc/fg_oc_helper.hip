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
//   others   for a block of kOcRows OUTPUT rows of M_not: row r of an object holds the vertex at walk position r + m(r),
//            m(r) = members met before the r-th non-member, a step function that M itself tells (member j at walk
//            position w_j comes before row r iff w_j - j <= r).  So nothing is walked: a lane keeps the next four steps
//            of each of its objects in registers and the rows are written with arithmetic alone.
// Lanes are objects throughout, so objects of one row split read neighbouring vertices; all objects of a wavefront that
// share a window read it through scalar loads (count, members).
// Integer-only; bound by the M_not write stream (n_unique x n_maxrs words).  10 x 100,000 vertices, 2,000 objects,
// 0.82 GB: 815 -> 395 us (count 100 -> 34, scan 56 -> 11, members 171 -> 50, others 509 -> 302, of which the stores
// alone would take some 160).
// Without a workspace the single-kernel form of the paper is used.
#include "fg_internal.hpp"

namespace fg {

constexpr int kOcBlock = 64;
constexpr int kOcBatch = 8;       // independent loads kept in flight per lane
constexpr int kOcChunk = 128;     // walk positions per chunk, and output rows per block of the M_not kernel

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

// Rows r0 .. r1-1 of one object by walking its vertices: for objects with more members than rows in M, whose later
// members M does not tell.
__device__ __forceinline__ void oc_others_walk(const OcWindow& w, int32_t k, int32_t r0, int32_t r1, const int32_t* __restrict__ asso_idx,
                                               int32_t n_unique, int32_t n_chunks, const int32_t* __restrict__ counts,
                                               int32_t* __restrict__ M_not)
{
    // largest chunk c whose start has at most r0 non-members before it: c*C - members_before(c) <= r0
    int32_t lo = 0, hi = n_chunks;           // invariant: others_before(lo) <= r0; chunks >= hi are too far (or hi = n_chunks)
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        const int32_t before = mid * kOcChunk - counts[(int64_t)mid * n_unique + k];
        if (before <= r0) lo = mid; else hi = mid;
    }
    int32_t p = lo * kOcChunk;
    int32_t fill = p - counts[(int64_t)lo * n_unique + k];      // non-members before walk position p
    // phase 1, no stores: advance to the walk position where this object's non-member count reaches r0.
    // Lanes need different numbers of steps here; keeping it apart from the emission lets the emission
    // run with every lane at the same output row.
    while (p < w.len && fill < r0) {
        int32_t v[kOcBatch];
#pragma unroll
        for (int u = 0; u < kOcBatch; ++u) v[u] = p + u < w.len ? asso_idx[oc_vertex(w, p + u)] : w.uq;
        int32_t adv = 0;
#pragma unroll
        for (int u = 0; u < kOcBatch; ++u) {
            if (fill < r0) { fill += v[u] != w.uq; ++adv; }
        }
        p += adv;
    }
    // phase 2: emit rows r0 .. r1-1; a lane falls one row behind its neighbours only when it meets a member
    int32_t r = r0;
    while (p < w.len && r < r1) {
        int32_t v[kOcBatch];
#pragma unroll
        for (int u = 0; u < kOcBatch; ++u) v[u] = p + u < w.len ? asso_idx[oc_vertex(w, p + u)] : w.uq;   // past the end: skipped like a member
#pragma unroll
        for (int u = 0; u < kOcBatch; ++u) {
            if (v[u] != w.uq && r < r1) { M_not[(int64_t)r * n_unique + k] = oc_vertex(w, p + u); ++r; }
        }
        p += kOcBatch;
    }
    for (; r < r1; ++r) M_not[(int64_t)r * n_unique + k] = -1;
}

// One wavefront per 64 * VEC objects and kOcRows output rows of M_not; a lane has VEC neighbouring objects and writes
// them with one store a row (VEC = 4: 1 KB a wavefront and row; needs n_unique a multiple of four and M_not on a 16-byte
// boundary, else VEC = 1).
constexpr int kOcRows = 256;
constexpr int kOcSteps = 4;       // next steps of an object held in registers
template <int VEC>
__global__ void __launch_bounds__(kOcBlock)
k_oc_others(const int32_t* __restrict__ asso_idx, const int32_t* __restrict__ unique_idx,
            const int32_t* __restrict__ unique_rs_asso, const int32_t* __restrict__ rs, int32_t n_vert, int32_t n_unique,
            int32_t n_splits, int32_t n_maxuq, int32_t n_maxrs, int32_t rot_block, int32_t n_chunks,
            const int32_t* __restrict__ counts, const int32_t* __restrict__ M, int32_t* __restrict__ M_not)
{
    // n_unique is a multiple of VEC, so a lane's objects all exist or none does; lanes without any shadow the last ones
    // (the wavefront's minimum below takes every lane) and write nothing
    const int32_t at_k = (blockIdx.x * kOcBlock + threadIdx.x) * VEC;
    const bool mine = at_k < n_unique;
    const int32_t k0 = mine ? at_k : n_unique - VEC;
    const int32_t r0 = blockIdx.y * kOcRows;
    const int32_t r1 = r0 + kOcRows < n_maxrs ? r0 + kOcRows : n_maxrs;
    OcWindow w[VEC];
    int32_t total[VEC], j[VEC], step[VEC][kOcSteps];
    bool cut = false;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        w[i] = oc_window(k0 + i, unique_idx, unique_rs_asso, rs, n_vert, n_splits, n_maxrs, rot_block);
        total[i] = counts[(int64_t)n_chunks * n_unique + k0 + i];
        cut = cut || total[i] > n_maxuq;
        j[i] = 0;
    }
    if (__any(cut)) {
#pragma unroll 1
        for (int i = 0; i < VEC && mine; ++i) {
            const OcWindow wi = oc_window(k0 + i, unique_idx, unique_rs_asso, rs, n_vert, n_splits, n_maxrs, rot_block);
            oc_others_walk(wi, k0 + i, r0, r1, asso_idx, n_unique, n_chunks, counts, M_not);
        }
        return;
    }
    // the row from which on member q of object i lies behind: its walk position less the members before it
    auto row_of = [&](int i, int32_t q) -> int32_t {
        int32_t o = M[(int64_t)q * n_unique + k0 + i] - w[i].start - w[i].rot;
        if (o < 0) o += w[i].len;
        return o - q;
    };
    // moves every object past its members that lie before row r, then reads the next steps
    auto seek = [&](int32_t r, bool far) {
        if (far) {                                       // rows of the members ascend: halving
            int32_t hi[VEC];
#pragma unroll
            for (int i = 0; i < VEC; ++i) hi[i] = total[i];
            for (;;) {
                bool open = false;
#pragma unroll
                for (int i = 0; i < VEC; ++i) open = open || j[i] < hi[i];
                if (!__any(open)) break;
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    if (j[i] < hi[i]) {
                        const int32_t mid = (j[i] + hi[i]) >> 1;
                        if (row_of(i, mid) <= r) j[i] = mid + 1; else hi[i] = mid;
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i)
#pragma unroll
            for (int q = 0; q < kOcSteps; ++q) step[i][q] = j[i] + q < total[i] ? row_of(i, j[i] + q) : 0x7fffffff;
    };
    seek(r0, true);
    for (int32_t r = r0; r < r1;) {
        // the steps in registers hold up to the row where some object reaches its last one
        int32_t stop = r1;
#pragma unroll
        for (int i = 0; i < VEC; ++i) stop = step[i][kOcSteps - 1] < stop ? step[i][kOcSteps - 1] : stop;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t other = __shfl_xor(stop, o, 64);
            stop = other < stop ? other : stop;
        }
        stop = __builtin_amdgcn_readfirstlane(stop);
        for (; r < stop; ++r) {
            int32_t v[VEC];
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                int32_t p = r + j[i];
#pragma unroll
                for (int q = 0; q < kOcSteps - 1; ++q) p += r >= step[i][q];
                v[i] = p < w[i].len ? oc_vertex(w[i], p) : -1;
            }
            if (!mine) continue;
            int32_t* const at = M_not + (int64_t)r * n_unique + k0;
            if constexpr (VEC == 4) *reinterpret_cast<int4*>(at) = make_int4(v[0], v[1], v[2], v[3]);
            else at[0] = v[0];
        }
        if (r < r1) {
            bool far = false;
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                int32_t passed = 0;
#pragma unroll
                for (int q = 0; q < kOcSteps; ++q) passed += step[i][q] <= r;
                j[i] += passed;
                far = far || passed == kOcSteps;         // a run of members: there may be any number more of them
            }
            seek(r, __any(far));
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
        hipLaunchKernelGGL(k_oc_helper, dim3(groups), dim3(kOcBlock), 0, stream, asso_idx, unique_idx, unique_rs_asso, rs,
                           n_vert, n_unique, n_splits, n_maxuq, n_maxrs, calc_m_not, rot_block, M, M_not);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_oc_count, dim3(groups, n_chunks), dim3(kOcBlock), 0, stream, asso_idx, unique_idx, unique_rs_asso,
                       rs, n_vert, n_unique, n_splits, n_maxrs, rot_block, counts);
    hipLaunchKernelGGL(k_oc_scan, dim3(groups), dim3(kOcBlock * kOcScanWaves), 0, stream, counts, n_unique, n_chunks);
    int64_t pads = ((int64_t)n_maxuq + kOcPadRows - 1) / kOcPadRows;
    if (pads > 65535 - n_chunks) pads = 65535 - n_chunks;
    hipLaunchKernelGGL(k_oc_members, dim3(groups, n_chunks + (unsigned)pads), dim3(kOcBlock), 0, stream, asso_idx, unique_idx,
                       unique_rs_asso, rs, n_vert, n_unique, n_splits, n_maxuq, n_maxrs, rot_block, n_chunks, counts, M);
    if (calc_m_not) {
        const unsigned rows = (unsigned)((n_maxrs + (int64_t)kOcRows - 1) / kOcRows);
        if (n_unique % 4 == 0 && ((uintptr_t)M_not & 15) == 0)
            hipLaunchKernelGGL(k_oc_others<4>, dim3((groups + 3) / 4, rows), dim3(kOcBlock), 0, stream, asso_idx, unique_idx, unique_rs_asso,
                               rs, n_vert, n_unique, n_splits, n_maxuq, n_maxrs, rot_block, n_chunks, counts, M, M_not);
        else
            hipLaunchKernelGGL(k_oc_others<1>, dim3(groups, rows), dim3(kOcBlock), 0, stream, asso_idx, unique_idx, unique_rs_asso,
                               rs, n_vert, n_unique, n_splits, n_maxuq, n_maxrs, rot_block, n_chunks, counts, M, M_not);
    }
    return hipGetLastError();
}

}  // namespace fg
