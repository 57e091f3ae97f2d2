// Bounding boxes of the group kernel: leaves of 64 consecutive bin-ordered points, nodes of 64 leaves.
#pragma once
#include "fg_internal.hpp"

namespace fg {

constexpr int kGroupLeaf = 64;                  // points per leaf: one per lane

template <int D> constexpr int group_box_vecs() { return (2 * D + 3) / 4; }

// Boxes live in the work list's area (4 bytes a point): 80 bytes per 64 points and per 4096 points at most.
struct GroupTree { float4* leaf; float4* node; int32_t n_leaf, n_node; };

template <int D>
static __host__ __device__ __forceinline__ GroupTree group_tree(void* area, int32_t n)
{
    GroupTree t;
    t.n_leaf = (n + kGroupLeaf - 1) / kGroupLeaf;
    t.n_node = (t.n_leaf + 63) / 64;
    t.node = reinterpret_cast<float4*>(area);
    t.leaf = t.node + (size_t)t.n_node * group_box_vecs<D>();
    return t;
}

__device__ __forceinline__ float wave_min_f32(float v)
{
    const int id = __float_as_int(3.4028235e38f);
    auto step = [&](int o) { v = fminf(v, __int_as_float(o)); };
    step(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x111, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x112, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x114, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x118, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x142, 0xa, 0xf, false));
    step(__builtin_amdgcn_update_dpp(id, __float_as_int(v), 0x143, 0xc, 0xf, false));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Boxes of the 64 leaves of a node and its own, by a workgroup of WAVES wavefronts.  A wavefront requests the points of four leaves
// together.
template <int D, int WAVES>
__device__ __forceinline__ void group_boxes(const float4* __restrict__ rec, int32_t n, const GroupTree& tree, int32_t node)
{
    constexpr int NB = group_box_vecs<D>();
    __shared__ float red[WAVES][2 * D];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float m[2 * D];                               // minima of x and of -x
#pragma unroll
    for (int c = 0; c < 2 * D; ++c) m[c] = 3.4028235e38f;
#pragma unroll 1
    for (int i0 = 0; i0 < 64 / WAVES; i0 += 4) {
        const int32_t leaf0 = node * 64 + wv * (64 / WAVES) + i0;
        if (leaf0 >= tree.n_leaf) break;
        float x[4][D];
        int32_t row;
#pragma unroll
        for (int i = 0; i < 4; ++i) load_rec<D>(rec, min((leaf0 + i) * kGroupLeaf + lane, n - 1), x[i], row);      // past the end: the last point once more
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float w[NB * 4];
#pragma unroll
            for (int c = 0; c < NB * 4; ++c) w[c] = 0.0f;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const float mn = wave_min_f32(x[i][c]), mx = wave_min_f32(-x[i][c]);
                m[c] = fminf(m[c], mn);
                m[D + c] = fminf(m[D + c], mx);
                w[c] = mn;
                w[D + c] = -mx;
            }
            if (lane == 0 && leaf0 + i < tree.n_leaf) {
#pragma unroll
                for (int v = 0; v < NB; ++v) tree.leaf[(int64_t)(leaf0 + i) * NB + v] = make_float4(w[4 * v], w[4 * v + 1], w[4 * v + 2], w[4 * v + 3]);
            }
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < 2 * D; ++c) red[wv][c] = m[c];
    }
    __syncthreads();
    if (threadIdx.x < 2 * D) {
        const int c = threadIdx.x;
        float v = red[0][c];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v = fminf(v, red[w][c]);
        reinterpret_cast<float*>(tree.node + (int64_t)node * NB)[c] = c < D ? v : -v;
    }
}

// The same in two launches, where there is other work beside them: the box of a leaf by a wavefront, then that of a node.
template <int D>
__device__ __forceinline__ void group_leaf_box(const float4* __restrict__ rec, int32_t n, const GroupTree& tree, int32_t leaf)
{
    constexpr int NB = group_box_vecs<D>();
    const int lane = threadIdx.x & 63;
    float x[D], w[NB * 4];
    int32_t row;
    load_rec<D>(rec, min(leaf * kGroupLeaf + lane, n - 1), x, row);
#pragma unroll
    for (int c = 0; c < NB * 4; ++c) w[c] = 0.0f;
#pragma unroll
    for (int c = 0; c < D; ++c) {
        w[c] = wave_min_f32(x[c]);
        w[D + c] = -wave_min_f32(-x[c]);
    }
    if (lane == 0) {
#pragma unroll
        for (int v = 0; v < NB; ++v) tree.leaf[(int64_t)leaf * NB + v] = make_float4(w[4 * v], w[4 * v + 1], w[4 * v + 2], w[4 * v + 3]);
    }
}
template <int D>
__device__ __forceinline__ void group_node_box(const GroupTree& tree, int32_t node)
{
    constexpr int NB = group_box_vecs<D>();
    const int lane = threadIdx.x & 63;
    const int32_t leaf = min(node * 64 + lane, tree.n_leaf - 1);
    float w[NB * 4];
#pragma unroll
    for (int v = 0; v < NB; ++v) {
        const float4 f = tree.leaf[(int64_t)leaf * NB + v];
        w[4 * v] = f.x; w[4 * v + 1] = f.y; w[4 * v + 2] = f.z; w[4 * v + 3] = f.w;
    }
#pragma unroll
    for (int c = 0; c < D; ++c) {
        w[c] = wave_min_f32(w[c]);
        w[D + c] = -wave_min_f32(-w[D + c]);
    }
    if (lane == 0) {
#pragma unroll
        for (int v = 0; v < NB; ++v) tree.node[(int64_t)node * NB + v] = make_float4(w[4 * v], w[4 * v + 1], w[4 * v + 2], w[4 * v + 3]);
    }
}

}  // namespace fg
