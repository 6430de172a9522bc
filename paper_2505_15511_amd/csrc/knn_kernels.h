// Device kernels of the in-cluster exact nearest-neighbour index for gfx950 (Section 3.2 of arxiv 2505.15511: the
// candidates for a point's neighbours are the points of its own cluster; among those the neighbours are exact).
//
// A dense contraction: all pairwise dot products inside a cluster.  The stages:
//   k_knn_cells    long groups of wide rows only: the rows of a group in the order of cells (k_knn_place), near rows together;
//   k_knn_pack     every row centred, scaled by a power of two and split into two float16 parts, x' = hi + lo to 2^-22 of x',
//                  laid out tile by tile in the order the matrix instructions read their operands;
//   k_knn_filter   float16 matrix cores (hi hi + hi lo + lo hi, float32 accumulation): for every query the K' = k + pad
//                  candidates with the smallest key |c|^2 - 2 q.c, and tau (every point left out has key >= tau, but for those that
//                  another slice's distances rule out: these are farther than the K'-th nearest for certain);
//   k_knn_refine   sorts those candidates by (distance, index), distance = sum_t (x_t - y_t)^2 in float64 in the order
//                  t = 0..d-1, worked out where the filter's error bound leaves the order open; the first k are the answer
//                  if the k-th lies below tau by more than that bound -- otherwise the query is flagged;
//   k_knn_exact    flagged queries (near-ties beyond the pad, duplicates in bulk): exact distances to the whole cluster.
// The result therefore does not depend on the filter's rounding: it is the float64 definition, tie-broken by index.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "knn_filter_kernel.h"
#include "rows.h"

namespace nomad_knn {

// Distances do not change when a cluster is moved as a whole, and the float32 error of the filter grows with |x|^2:
// the filter therefore works on rows centred on their cluster, x' = fl(x - c_r), c_r = the mean in float32 of a sample of the cluster's
// rows: any centre gives the same answers, and one that 256 rows and more give is off by a sixteenth of the rows' deviation
// (|x'|^2, and with it the bound, by 1/256).  One row of every `centre_step`, a different one of each so that rows in a periodic order are met too.
// 1,000,000 x 128: all rows 100 us (one cluster) and 103 (six slices), the sample 31 and 12 (the atomics
// on one cluster's words); 100,003 x 768, the points and 64 clusters: 124 -> 77.
__host__ __device__ inline uint32_t centre_step(uint32_t rows) { return rows >= 4096u ? 16u : rows >= 2048u ? 8u : rows >= 1024u ? 4u : rows >= 512u ? 2u : 1u; }
// Column sums of a cluster, a slab of rows per block, one thread per column.  Slabs are cut so that there are a few for every
// compute unit (3,001 x 50: three slabs of 1,024 rows took 38 us; 100,003 x 768: 98 of them 191 us), 32 to 1,024 rows.
inline int32_t centroid_rows(int64_t n) {
    int32_t rows = 32;
    while (rows < 1024 && n / rows > 1024) rows *= 2;
    return rows;
}
__global__ void __launch_bounds__(256) k_knn_centroid_sums(const float* __restrict__ X, int32_t d, const int32_t* __restrict__ members,
                                                           const uint32_t* __restrict__ start, const KnnBlock* __restrict__ slabs,
                                                           int32_t rows, float* __restrict__ centre) {
    const KnnBlock sl = slabs[blockIdx.x];   // rows q0 .. q0 + rows of cluster sl.cluster
    const uint32_t c0 = start[sl.cluster], n_g = start[sl.cluster + 1] - c0, step = centre_step(n_g);
    const uint32_t q1 = min(n_g, (uint32_t)(sl.q0 + rows));
    const auto sums = [&](uint32_t b0, uint32_t b1, const auto& position) {
        for (int col = threadIdx.x; col < d; col += 256) {
            float s = 0.f;
            uint32_t b = b0;
            for (; b + 16 <= b1; b += 16) {   // sixteen rows in flight
                int32_t row[16];
                float v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) row[u] = knn_row(members, position(b + u));
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = X[(int64_t)row[u] * d + col];
#pragma unroll
                for (int u = 0; u < 16; ++u) s += v[u];
            }
            for (; b < b1; ++b) s += X[(int64_t)knn_row(members, position(b)) * d + col];
            atomicAdd(&centre[(int64_t)sl.cluster * d + col], s);
        }
    };
    // (short clusters, all rows: a loop of their own, 400,000 x 16 in clusters of 200 31 -> 25 us)
    if (step == 1u) sums((uint32_t)sl.q0, q1, [&](uint32_t b) { return c0 + b; });
    else sums((uint32_t)sl.q0 / step, (q1 + step - 1) / step, [&](uint32_t b) { return c0 + min(b * step + (b * 0x9E3779B1u >> 28 & (step - 1u)), n_g - 1u); });   // (slabs are whole steps)
}
__global__ void __launch_bounds__(256) k_knn_centroid_finish(float* __restrict__ centre, const uint32_t* __restrict__ start, int32_t R, int32_t d) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= (int64_t)R * d) return;
    const int32_t r = (int32_t)(x / d);
    const uint32_t n_g = start[r + 1] - start[r], cnt = (n_g + centre_step(n_g) - 1) / centre_step(n_g);
    centre[x] = cnt ? centre[x] / (float)cnt : 0.f;
}

// |x'|^2 of every centred row in float32 and the largest one per cluster.  Sixteen lanes share a row (a wavefront reads
// four consecutive rows, each lane every sixteenth column or 16-byte chunk) and add their partial sums pairwise: at most 4 ceil(d / 64)
// additions one after the other and four pairwise ones, which is what knn_filter_eps allows the norm for.  Bound by the latency of two
// or three loads in a chain and, where the groups are few, by the atomics on their words: large sets take kNormBatch rows per
// sixteen lanes, all their loads in flight, and one atomic per workgroup that lies inside one group.  `members` lists the rows
// group by group where the caller has that order: the centres then come from the first cache.  1,000,000 x 128: one group 175 ->
// 84 us (6.1 TB/s), six slices 290 -> 85, 256 clusters of mixed rows 175 -> 155.
static_assert(kNormLanes == 16, "four pairwise additions");
constexpr int kNormRows = 256 / kNormLanes;   // rows per workgroup and batch entry
constexpr int kNormBatch = 4, kNormBatches = 4;
// batches of a workgroup: as many as leave 2,048 of them; 0: one row per sixteen lanes, where batches would leave units without work
inline int norm_batches(int64_t n) { return n < 65536 ? 0 : n < ((int64_t)1 << 18) ? 1 : n < ((int64_t)1 << 19) ? 2 : kNormBatches; }
inline int64_t norm_block_rows(int64_t n) { return (int64_t)kNormRows * (norm_batches(n) ? kNormBatch * norm_batches(n) : 1); }

// U rows of sixteen lanes each, i0 + u stride: their sums, of rows that are none zero
template <int U>
__device__ __forceinline__ void centred_norms(const float* __restrict__ X, int64_t n, int32_t d, const int32_t* __restrict__ members,
                                              const int32_t* __restrict__ cluster_of, const float* __restrict__ centre, int64_t i0, int64_t stride,
                                              int part, int32_t* row, int32_t* g, float* s) {
    const float *x[U], *c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) row[u] = knn_row(members, (uint32_t)(i0 + u * stride < n ? i0 + u * stride : n - 1));
#pragma unroll
    for (int u = 0; u < U; ++u) {
        x[u] = X + (int64_t)row[u] * d;
        g[u] = cluster_of ? cluster_of[row[u]] : 0;
        s[u] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = centre + (int64_t)g[u] * d;
    if (rows_by_16(X, d)) {   // (the centres are the library's own, see knn.hip)
        for (int t = 4 * part; t < d; t += 4 * kNormLanes) {
            float4 xv[U], cv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) { xv[u] = *(const float4*)(x[u] + t); cv[u] = *(const float4*)(c[u] + t); }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float v = xv[u].x - cv[u].x;
                s[u] = fmaf(v, v, s[u]);
                v = xv[u].y - cv[u].y;
                s[u] = fmaf(v, v, s[u]);
                v = xv[u].z - cv[u].z;
                s[u] = fmaf(v, v, s[u]);
                v = xv[u].w - cv[u].w;
                s[u] = fmaf(v, v, s[u]);
            }
        }
    } else {
        for (int t = part; t < d; t += kNormLanes) {
            float xv[U], cv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) { xv[u] = x[u][t]; cv[u] = c[u][t]; }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float v = xv[u] - cv[u];
                s[u] = fmaf(v, v, s[u]);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        for (int w = kNormLanes / 2; w > 0; w >>= 1) s[u] += __shfl_xor(s[u], w, kNormLanes);   // every lane of the row: the row's sum
        if (i0 + u * stride >= n) s[u] = 0.f;
    }
}
// non-negative floats order like their bit patterns; the maximum only grows: a stale read costs one atomic, not the result
__device__ __forceinline__ void raise_norm(uint32_t* __restrict__ word, uint32_t bits) {
    if (bits > *word) atomicMax(word, bits);
}
__global__ void __launch_bounds__(256) k_knn_norms(const float* __restrict__ X, int64_t n, int32_t d, const int32_t* __restrict__ members,
                                                   const int32_t* __restrict__ cluster_of, const float* __restrict__ centre, float* __restrict__ norm,
                                                   uint32_t* __restrict__ max_norm_bits, int32_t batches) {
    __shared__ int32_t group[4];
    __shared__ uint32_t most[4];
    const int part = threadIdx.x % kNormLanes;
    const int64_t row = threadIdx.x / kNormLanes;
    int32_t cur = -1;          // the group that `bits` is the maximum of
    uint32_t bits = 0u;
    const auto enter = [&](int64_t i, int32_t r, int32_t g, float s) {
        if (i >= n) return;
        if (part == 0 && norm) norm[r] = s;
        if (g != cur) {
            if (cur >= 0 && part == 0) raise_norm(&max_norm_bits[cur], bits);
            cur = g;
            bits = 0u;
        }
        bits = max(bits, __float_as_uint(s));
    };
    if (batches == 0) {
        const int64_t i = (int64_t)blockIdx.x * kNormRows + row;
        int32_t r[1], g[1];
        float s[1];
        centred_norms<1>(X, n, d, members, cluster_of, centre, i, 0, part, r, g, s);
        enter(i, r[0], g[0], s[0]);
    } else {
        for (int b = 0; b < batches; ++b) {
            const int64_t i = ((int64_t)blockIdx.x * batches + b) * (kNormRows * kNormBatch) + row;
            int32_t r[kNormBatch], g[kNormBatch];
            float s[kNormBatch];
            centred_norms<kNormBatch>(X, n, d, members, cluster_of, centre, i, kNormRows, part, r, g, s);
#pragma unroll
            for (int u = 0; u < kNormBatch; ++u) enter(i + u * kNormRows, r[u], g[u], s[u]);
        }
    }
    // the wavefront's own group, or -1 where it has several (those go out by themselves) or none
    const unsigned long long live = __ballot(cur >= 0);
    const int32_t g0 = live ? __shfl(cur, __ffsll((long long)live) - 1, 64) : -1;
    const bool one = __all(cur < 0 || cur == g0);
    for (int w = 32; w >= kNormLanes && one; w >>= 1) bits = max(bits, (uint32_t)__shfl_xor((int)bits, w, 64));
    if (!one && cur >= 0 && part == 0) raise_norm(&max_norm_bits[cur], bits);
    if ((threadIdx.x & 63) == 0) { group[threadIdx.x >> 6] = one ? g0 : -1; most[threadIdx.x >> 6] = bits; }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int32_t own = group[threadIdx.x];
        uint32_t m = 0u;
        bool first = own >= 0;
        for (int w = 0; w < 4; ++w)
            if (group[w] == own) { m = max(m, most[w]); first = first && w >= (int)threadIdx.x; }
        if (first) raise_norm(&max_norm_bits[own], m);
    }
}

// cluster sizes; a block counts kCountSpan labels in LDS first where the clusters are few enough to fit there
constexpr int kCountSpan = 16384;
constexpr int kCountLds = 4096;
__global__ void __launch_bounds__(256) k_knn_count(const int32_t* __restrict__ cluster_of, int64_t n, int32_t R, uint32_t* __restrict__ counts,
                                                   int* __restrict__ bad) {
    __shared__ uint32_t h[kCountLds];
    const bool local = R <= kCountLds;
    if (local) {
        for (int r = threadIdx.x; r < R; r += 256) h[r] = 0u;
        __syncthreads();
    }
    const int64_t i0 = (int64_t)blockIdx.x * kCountSpan, i1 = min(n, i0 + kCountSpan);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const int32_t r = cluster_of[i];
        if (r < 0 || r >= R) { *bad = 1; continue; }
        if (local) atomicAdd(&h[r], 1u);
        else atomicAdd(&counts[r], 1u);
    }
    if (local) {
        __syncthreads();
        for (int r = threadIdx.x; r < R; r += 256)
            if (h[r]) atomicAdd(&counts[r], h[r]);
    }
}

// members grouped by cluster (any order inside a cluster: ties are broken by the point index, not by position).  A
// workgroup takes kGroupSpan points: ranks inside the workgroup from an LDS counter per cluster, then one global
// reservation per cluster it met (clusters beyond kCountLds: one global atomic per point).
constexpr int kGroupSpan = 4096;
__global__ void __launch_bounds__(256) k_knn_group(const int32_t* __restrict__ cluster_of, int64_t n, int32_t R, const uint32_t* __restrict__ start,
                                                   uint32_t* __restrict__ cursor, int32_t* __restrict__ members) {
    __shared__ uint32_t h[kCountLds];     // count, then global base, of every cluster inside this workgroup's span
    const int64_t i0 = (int64_t)blockIdx.x * kGroupSpan;
    constexpr int kPer = kGroupSpan / 256;
    if (R > kCountLds) {
        for (int u = 0; u < kPer; ++u) {
            const int64_t i = i0 + u * 256 + threadIdx.x;
            if (i < n) { const int32_t r = cluster_of[i]; members[start[r] + atomicAdd(&cursor[r], 1u)] = (int32_t)i; }
        }
        return;
    }
    for (int r = threadIdx.x; r < R; r += 256) h[r] = 0u;
    __syncthreads();
    int32_t cl[kPer];
    uint32_t rk[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int64_t i = i0 + u * 256 + threadIdx.x;
        cl[u] = i < n ? cluster_of[i] : -1;
        rk[u] = cl[u] >= 0 ? atomicAdd(&h[cl[u]], 1u) : 0u;
    }
    __syncthreads();
    for (int r = threadIdx.x; r < R; r += 256)
        if (h[r]) h[r] = start[r] + atomicAdd(&cursor[r], h[r]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (cl[u] >= 0) members[h[cl[u]] + rk[u]] = (int32_t)(i0 + u * 256 + threadIdx.x);
}

// ---------------------------------------------------------------- the order of the rows inside a group
// The filter passes over a tile of candidates after a third of its products where none of them can be among the nearest of any of the
// tile's queries.  In random order hardly a tile of a short group is so; where the rows of a group lie cell by cell, most are, as far as
// the rows of a group differ by more than noise.  A group's cells are the nearest of kCells of its rows.  The order has no part in the answers.
constexpr int kCells = 16;
// Mean rows of a group times columns from which the filter gains more than the order costs (the cells' products beside the norms, 0.05 ms
// for 1,000,000 x 128, and two launches).  Mixtures with four components a cluster, k = 10 to 32, calls without and with the order: clusters of 500 x 128
// 1.18 / 1.26 to 2.13 / 2.27 ms, 500 x 250 2.32 / 2.35 to 3.46 / 3.41, 500 x 400 1.15 / 1.11, 1,500 x 64 1.54 / 1.55 to 2.66 / 2.81,
// 1,500 x 128 1.63 / 1.55 to 2.80 / 2.84, 4,000 x 30 2.04 / 1.90 to 3.43 / 3.54, 4,000 x 64 2.34 / 2.12 to 3.87 / 3.71, 4,000 x 256 2.72 / 2.29 to 4.28 / 3.59;
// isotropic rows, which have no cells worth the name: 3,900 x 128 5.86 / 5.99.
// Long lists in 32-row tiles take their longest from the queries' own tiles, which come first: where all workgroups run at once nothing makes up for it.  k = 30, clusters of
// 4,000 x 64 and 2,000 x 120, unordered / ordered: 33,000 points 0.44 / 0.48 and 0.41 / 0.45 ms, 50,000 0.44 / 0.50 and 0.43 / 0.47, 70,000 0.74 / 0.68 and 0.66 / 0.65, 200,000 1.41 / 1.22 and 1.25 / 1.17.
inline bool knn_ordered(int64_t n, int32_t d, int32_t groups, int32_t list_len) {
    return n * d >= (int64_t)200000 * groups && (n > 65536 || list_len <= kShortList || knn_tile(d, list_len) == 16);
}

// the sum over the sixteen lanes of a row of lanes, in all of them
template <int CTRL> __device__ __forceinline__ float add_lanes(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float sum_of_16(float v) { return add_lanes<0x140>(add_lanes<0x141>(add_lanes<0x4E>(add_lanes<0xB1>(v)))); }

// k_knn_norms for rows in the order of their groups, with the cell of every row, and how many of the group each cell has.  A slab of a group's rows
// per workgroup, its cells' rows in LDS.  Bound by the one read of the rows and, nearly as much, the vector pipe: 1,000,000 x 128 0.20 ms, the
// norms alone 0.16.
__global__ void __launch_bounds__(256) k_knn_cells(const float* __restrict__ X, int32_t d, const int32_t* __restrict__ members, const uint32_t* __restrict__ start,
                                                   const KnnBlock* __restrict__ slabs, int32_t rows, const float* __restrict__ centre, float* __restrict__ norm,
                                                   uint32_t* __restrict__ max_norm_bits, uint8_t* __restrict__ cell_of, uint32_t* __restrict__ counts) {
    extern __shared__ float4 lds_pivots[];     // [kCells][width / 4] rows, then the centre's
    __shared__ float half_norm[kCells];
    __shared__ uint32_t hist[kCells], most;
    const KnnBlock sl = slabs[blockIdx.x];
    const uint32_t c0 = start[sl.cluster], n_g = start[sl.cluster + 1] - c0;
    const uint32_t r0 = c0 + (uint32_t)sl.q0, r1 = min(c0 + n_g, r0 + (uint32_t)rows);
    const int width = (d + 3) / 4 * 4, part = threadIdx.x % kNormLanes, mine = threadIdx.x / kNormLanes;
    float* const pivots = (float*)lds_pivots;
    float* const middle = pivots + kCells * width;
    if (threadIdx.x < kCells) hist[threadIdx.x] = 0u;
    if (threadIdx.x == 0) most = 0u;
    for (int t = threadIdx.x; t < width; t += 256) middle[t] = t < d ? centre[(int64_t)sl.cluster * d + t] : 0.f;
    __syncthreads();
    {   // (kCells = 256 / kNormLanes: sixteen lanes a row)
        const float* x = X + (int64_t)knn_row(members, c0 + (uint32_t)((uint64_t)n_g * (uint32_t)mine / kCells)) * d;
        float s = 0.f;
        for (int t = part; t < width; t += kNormLanes) {
            const float v = t < d ? x[t] - middle[t] : 0.f;
            pivots[mine * width + t] = v;
            s = fmaf(v, v, s);
        }
        s = sum_of_16(s);
        if (part == 0) half_norm[mine] = 0.5f * s;
    }
    __syncthreads();
    const bool vec = rows_by_16(X, d);
    uint32_t bits = 0u;
    for (uint32_t i0 = r0 + (uint32_t)mine; i0 - (uint32_t)mine < r1; i0 += kNormRows * kNormBatch) {
        int32_t row[kNormBatch];
        const float* x[kNormBatch];
        float s[kNormBatch], dot[kNormBatch][kCells];
#pragma unroll
        for (int u = 0; u < kNormBatch; ++u) row[u] = members[min(i0 + u * kNormRows, r1 - 1u)];
#pragma unroll
        for (int u = 0; u < kNormBatch; ++u) {
            x[u] = X + (int64_t)row[u] * d;
            s[u] = 0.f;
#pragma unroll
            for (int p = 0; p < kCells; ++p) dot[u][p] = 0.f;
        }
        if (vec) {
            for (int t = 4 * part; t < d; t += 4 * kNormLanes) {
                float4 v[kNormBatch];
#pragma unroll
                for (int u = 0; u < kNormBatch; ++u) v[u] = *(const float4*)(x[u] + t);
                const float4 c = *(const float4*)(middle + t);
#pragma unroll
                for (int u = 0; u < kNormBatch; ++u) {
                    v[u].x -= c.x; v[u].y -= c.y; v[u].z -= c.z; v[u].w -= c.w;
                    s[u] = fmaf(v[u].w, v[u].w, fmaf(v[u].z, v[u].z, fmaf(v[u].y, v[u].y, fmaf(v[u].x, v[u].x, s[u]))));
                }
#pragma unroll
                for (int p = 0; p < kCells; ++p) {
                    const float4 y = *(const float4*)(pivots + p * width + t);
#pragma unroll
                    for (int u = 0; u < kNormBatch; ++u) dot[u][p] = fmaf(v[u].w, y.w, fmaf(v[u].z, y.z, fmaf(v[u].y, y.y, fmaf(v[u].x, y.x, dot[u][p]))));
                }
            }
        } else {
            for (int t = part; t < d; t += kNormLanes) {
                float v[kNormBatch];
#pragma unroll
                for (int u = 0; u < kNormBatch; ++u) v[u] = x[u][t];
#pragma unroll
                for (int u = 0; u < kNormBatch; ++u) {
                    v[u] -= middle[t];
                    s[u] = fmaf(v[u], v[u], s[u]);
                }
#pragma unroll
                for (int p = 0; p < kCells; ++p) {
                    const float y = pivots[p * width + t];
#pragma unroll
                    for (int u = 0; u < kNormBatch; ++u) dot[u][p] = fmaf(v[u], y, dot[u][p]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kNormBatch; ++u) {
            s[u] = sum_of_16(s[u]);
            float best = 0.f;
            int cell = 0;
#pragma unroll
            for (int p = 0; p < kCells; ++p) {
                const float key = half_norm[p] - sum_of_16(dot[u][p]);
                if (p == 0 || key < best) { best = key; cell = p; }
            }
            const uint32_t i = i0 + u * kNormRows;
            if (part == 0 && i < r1) {
                norm[row[u]] = s[u];
                cell_of[i] = (uint8_t)cell;
                atomicAdd(&hist[cell], 1u);
                bits = max(bits, __float_as_uint(s[u]));
            }
        }
    }
    atomicMax(&most, bits);
    __syncthreads();
    if (threadIdx.x < kCells && hist[threadIdx.x]) atomicAdd(&counts[(size_t)sl.cluster * kCells + threadIdx.x], hist[threadIdx.x]);
    if (threadIdx.x == 0) raise_norm(&max_norm_bits[sl.cluster], most);
}

// the members of every group cell by cell; cursor [groups][kCells] begins at zero
__global__ void __launch_bounds__(256) k_knn_place(const int32_t* __restrict__ members, const uint8_t* __restrict__ cell_of, const uint32_t* __restrict__ start,
                                                   const KnnBlock* __restrict__ slabs, int32_t rows, const uint32_t* __restrict__ counts,
                                                   uint32_t* __restrict__ cursor, int32_t* __restrict__ out) {
    __shared__ uint32_t hist[kCells], base[kCells];
    const KnnBlock sl = slabs[blockIdx.x];
    const uint32_t c0 = start[sl.cluster], c1 = start[sl.cluster + 1];
    const uint32_t r0 = c0 + (uint32_t)sl.q0, r1 = min(c1, r0 + (uint32_t)rows);
    if (threadIdx.x < kCells) hist[threadIdx.x] = 0u;
    __syncthreads();
    constexpr int kPer = 4;                    // (slabs have up to 1,024 rows)
    uint32_t cell[kPer], rank[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const uint32_t i = r0 + u * 256 + threadIdx.x;
        cell[u] = i < r1 ? cell_of[i] : 0u;
        rank[u] = i < r1 ? atomicAdd(&hist[cell[u]], 1u) : 0u;
    }
    __syncthreads();
    if (threadIdx.x < kCells) {
        uint32_t before = c0;
        for (int p = 0; p < (int)threadIdx.x; ++p) before += counts[(size_t)sl.cluster * kCells + p];
        base[threadIdx.x] = before + atomicAdd(&cursor[(size_t)sl.cluster * kCells + threadIdx.x], hist[threadIdx.x]);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const uint32_t i = r0 + u * 256 + threadIdx.x;
        if (i < r1) out[base[cell[u]] + rank[u]] = members[i];
    }
}

// ---------------------------------------------------------------- stage 0: rows for the matrix cores
// Packs one tile of rows (positions pos0 .. of the n_g that begin at r0): a thread takes eight columns of one row at a time
// (adjacent threads adjacent rows: 16-byte stores side by side, the rows' lines shared inside the workgroup).  data: the tile's.
__device__ __forceinline__ void pack_tile(const float* __restrict__ X, int32_t d, const int32_t* __restrict__ members, uint32_t r0, uint32_t n_g, uint32_t pos0,
                                          const float* __restrict__ c, float scale, int32_t tile, int32_t steps, uint4* __restrict__ data) {
    const int tshift = tile == 32 ? 5 : 4, per_step = 64 >> tshift;   // chunks of eight columns per step
    const bool vec = rows_by_16(X, d);
    for (int x = threadIdx.x; x < (steps * 64); x += (int)blockDim.x) {
        const int row = x & (tile - 1), chunk = x >> tshift, col = 8 * chunk;
        const uint32_t pos = pos0 + (uint32_t)row;
        const bool live = pos < n_g;
        const float* src = X + (live ? (int64_t)knn_row(members, r0 + pos) : 0) * d;
        float v[8];
        if (vec) {
#pragma unroll
            for (int h = 0; h < 8; h += 4) {
                float4 a = make_float4(0.f, 0.f, 0.f, 0.f), m = a;
                if (live && col + h < d) { a = *(const float4*)(src + col + h); m = *(const float4*)(c + col + h); }
                v[h] = a.x - m.x; v[h + 1] = a.y - m.y; v[h + 2] = a.z - m.z; v[h + 3] = a.w - m.w;
            }
        } else {
#pragma unroll
            for (int h = 0; h < 8; ++h) v[h] = live && col + h < d ? src[col + h] - c[col + h] : 0.f;
        }
        half8 vh, vl;
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            const float y = v[h] * scale;
            vh[h] = (_Float16)y;
            vl[h] = (_Float16)(y - (float)vh[h]);
        }
        const int step = chunk / per_step, l = ((chunk % per_step) << tshift) + row;
        uint4* dst = data + (size_t)step * 128 + l;
        dst[0] = *(const uint4*)&vh;
        dst[64] = *(const uint4*)&vl;
    }
}

// the rows of a set, one workgroup per tile
__global__ void __launch_bounds__(256) k_knn_pack(const float* __restrict__ X, int32_t d, const int32_t* __restrict__ members,
                                                  const uint32_t* __restrict__ start, const uint32_t* __restrict__ tstart, int32_t groups,
                                                  const float* __restrict__ centre, const uint32_t* __restrict__ max_bits,
                                                  const uint32_t* __restrict__ other_bits, const float* __restrict__ row_norm, int32_t tile, int32_t steps, uint4* __restrict__ data,
                                                  float* __restrict__ norm) {
    const uint32_t t = blockIdx.x;
    int32_t g = 0, hi = groups;      // the group of this tile
    while (hi - g > 1) {
        const int32_t mid = (g + hi) >> 1;
        if (tstart[mid] <= t) g = mid; else hi = mid;
    }
    const uint32_t r0 = start[g], n_g = start[g + 1] - r0, pos0 = (t - tstart[g]) * (uint32_t)tile;
    pack_tile(X, d, members, r0, n_g, pos0, centre + (int64_t)g * d, ldexpf(1.f, knn_scale_exponent(max_bits[g])), tile, steps,
              data + (size_t)t * steps * 128);
    if (norm && threadIdx.x < (uint32_t)tile) {
        const uint32_t pos = pos0 + threadIdx.x;
        const float half_unit = ldexpf(0.5f, knn_scale_exponent(max_bits[g]) + knn_scale_exponent(other_bits[g]));
        norm[(size_t)t * tile + threadIdx.x] = pos < n_g ? row_norm[knn_row(members, r0 + pos)] * half_unit : __builtin_inff();
    }
}

// What an E step of Lloyd's iterations starts with, one workgroup per tile of centroids: the words that count from zero, the
// centroids' norms (kNormLanes sums a row, as in k_knn_norms) and the largest of them, the packed tile, and the copy the inertia
// is computed from.  Every workgroup reads all K rows for the largest norm, so this is for few and short ones (prepare_in_one_launch);
// beyond, the norms, the packing, the clearing and the copy are launches of their own (four of 3 to 4 us and their gaps; one of 5).
__global__ void __launch_bounds__(1024) k_kmeans_prepare(const float* __restrict__ C, int32_t K, int32_t d, const float* __restrict__ centre,
                                                        const uint32_t* __restrict__ point_bits, int32_t tile, int32_t steps, uint4* __restrict__ data,
                                                        float* __restrict__ norm, float* __restrict__ c_used, uint32_t* __restrict__ zeros, int32_t n_zeros,
                                                        uint32_t* __restrict__ max_cen) {
    __shared__ float own[32];          // |c'|^2 of this tile's rows
    __shared__ uint32_t largest;
    const uint32_t pos0 = blockIdx.x * (uint32_t)tile;
    if (threadIdx.x == 0) largest = 0u;
    if (threadIdx.x < 32u) own[threadIdx.x] = 0.f;
    __syncthreads();
    const int part = threadIdx.x % kNormLanes;
    uint32_t bits = 0u;
    for (int32_t r = threadIdx.x / kNormLanes; r < K; r += 1024 / kNormLanes) {
        float s = 0.f;
        for (int t = part; t < d; t += 8 * kNormLanes) {   // eight values in flight
            float x[8], c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) { const int at = min(t + u * kNormLanes, d - 1); x[u] = C[(int64_t)r * d + at]; c[u] = centre[at]; }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float v = t + u * kNormLanes < d ? x[u] - c[u] : 0.f;
                s = fmaf(v, v, s);
            }
        }
        for (int w = kNormLanes / 2; w > 0; w >>= 1) s += __shfl_xor(s, w, kNormLanes);
        bits = max(bits, __float_as_uint(s));
        if (part == 0 && (uint32_t)r >= pos0 && (uint32_t)r < pos0 + (uint32_t)tile) own[(uint32_t)r - pos0] = s;
    }
    atomicMax(&largest, bits);
    __syncthreads();
    const uint32_t top = largest;
    pack_tile(C, d, nullptr, 0u, (uint32_t)K, pos0, centre, ldexpf(1.f, knn_scale_exponent(top)), tile, steps, data + (size_t)blockIdx.x * steps * 128);
    if (threadIdx.x < (uint32_t)tile) {
        const float half_unit = ldexpf(0.5f, knn_scale_exponent(top) + knn_scale_exponent(point_bits[0]));
        norm[(size_t)blockIdx.x * tile + threadIdx.x] = pos0 + threadIdx.x < (uint32_t)K ? own[threadIdx.x] * half_unit : __builtin_inff();
    }
    const int64_t v0 = (int64_t)pos0 * d, v1 = min((int64_t)K * d, v0 + (int64_t)tile * d);
    for (int64_t v = v0 + threadIdx.x; v < v1; v += 1024) c_used[v] = C[v];
    if (blockIdx.x == 0) {
        if (threadIdx.x < (uint32_t)n_zeros) zeros[threadIdx.x] = 0u;
        if (threadIdx.x == 0) *max_cen = top;
    }
}

// the oracle's distance: difference, product and running sum each rounded once, in float64, t = 0..d-1 in order
// (by16: rows_by_16 of both sides' arrays)
__device__ __forceinline__ double exact_distance(const float* __restrict__ x, const float* __restrict__ y, int32_t d, bool by16) {
    double acc = 0.0;
    int t = 0;
    if (by16) {   // four values per load, still added one by one in order
        for (; t + 16 <= d; t += 16) {   // eight loads in flight before the first dependent addition
            float4 a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { a[u] = *(const float4*)(x + t + 4 * u); b[u] = *(const float4*)(y + t + 4 * u); }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                double diff = (double)a[u].x - (double)b[u].x;
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                diff = (double)a[u].y - (double)b[u].y;
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                diff = (double)a[u].z - (double)b[u].z;
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                diff = (double)a[u].w - (double)b[u].w;
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
            }
        }
        for (; t < d; t += 4) {
            const float4 a = *(const float4*)(x + t), b = *(const float4*)(y + t);
            double diff = (double)a.x - (double)b.x;
            acc = __dadd_rn(acc, __dmul_rn(diff, diff));
            diff = (double)a.y - (double)b.y;
            acc = __dadd_rn(acc, __dmul_rn(diff, diff));
            diff = (double)a.z - (double)b.z;
            acc = __dadd_rn(acc, __dmul_rn(diff, diff));
            diff = (double)a.w - (double)b.w;
            acc = __dadd_rn(acc, __dmul_rn(diff, diff));
        }
        return acc;
    }
    for (; t < d; ++t) {
        const double diff = (double)x[t] - (double)y[t];
        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
    }
    return acc;
}

// ---------------------------------------------------------------- stage 2: the order of the candidates
// The candidates arrive in the order of their filter keys.  Where a key lies below the next by more than twice the filter's
// error bound the exact distances stand in that order too; only the members of a run of closer keys need their exact
// distances to be ordered (by distance, then point), and of those only the runs that begin among the first k.  The
// kernel is bound by the rows it gathers: a million queries with 23 candidates of 128 columns, all exact, took 2.0 ms
// (5.9 TB/s out of the caches); with those whose order the bound leaves open 0.91 ms when the filter's sums were whole
// rows, 0.74 with sums of 64 columns and half the bound (100,003 x 768: a tenth of it, 0.79 -> 0.51).
// Certified, i.e. no point that the filter left out (key >= tau, exact key >= tau - eps) is nearer than the k-th, when the
// k-th key lies below tau by more than twice the bound (k candidates have exact keys up to key + eps), or else the k-th
// exact key, D_k - |q|^2, does by more than the bound; otherwise the query is flagged.  So is every query of a group that the
// filter cannot work on.
// G lanes per query (16, 32 or 64, at least the list length), one per candidate: short lists share a wavefront.
template <int G>
__global__ void __launch_bounds__(256) k_knn_refine(const KnnSets P, const int32_t* __restrict__ cand, const float* __restrict__ keys,
                                                    const float* __restrict__ tau, int32_t k, int32_t list_len, int32_t* __restrict__ out,
                                                    int32_t* __restrict__ flagged, uint32_t* __restrict__ n_flagged) {
    const int64_t p = (int64_t)blockIdx.x * (256 / G) + (threadIdx.x / G);   // position in the grouped query order
    const int lane = threadIdx.x % G;
    const int32_t d = P.d;
    if (p >= P.n_q) return;
    int32_t q = knn_row(P.qmembers, (uint32_t)p);
    if (G == 64) q = __builtin_amdgcn_readfirstlane(q);   // the same for the whole wavefront
    const float* xq = P.XQ + (int64_t)q * d;
    int32_t c = lane < list_len ? cand[p * list_len + lane] : -1;
    if (c >= P.n_c) c = -1;   // never an address outside the candidate rows, whatever the list holds
    const double key = c >= 0 ? (double)keys[p * list_len + lane] : __builtin_inf();
    const float t = tau[p];
    const int32_t g = P.group_of_q ? P.group_of_q[q] : 0;
    if (!knn_filter_usable(P.Q.max_bits[g], P.C.max_bits[g])) {   // the same for every lane of the query
        if (lane == 0) flagged[atomicAdd(n_flagged, 1u)] = q;
        return;
    }
    const double eps = knn_filter_eps(d, fmax((double)__uint_as_float(P.Q.max_bits[g]), (double)__uint_as_float(P.C.max_bits[g])), P.chunk);
    const int first = (int)(threadIdx.x & 63u) - lane;   // of this query's lanes in the wavefront
    const auto votes = [&](bool v) { return (__ballot(v) >> first) & (~0ull >> (64 - G)); };
    const double next = __shfl_down(key, 1, G);
    const int cnt = __popcll(votes(c >= 0));
    // (negated comparisons: a key that is not a number counts as close to everything)
    const unsigned long long links = votes(lane + 1 < cnt && !(next - key > 2.0 * eps));
    const unsigned long long breaks = ~links & ((1ull << lane) - 1ull);
    const int run0 = breaks ? 64 - __clzll((long long)breaks) : 0, run1 = lane + __ffsll((long long)(~links >> lane)) - 1;   // this lane's run
    const bool left_out = t < __builtin_inff() && cnt >= k;   // the same for every lane of the group
    const bool open = left_out && votes(lane == k - 1 && !(key + 2.0 * eps < (double)t)) != 0ull;
    const bool exact = c >= 0 && ((run1 > run0 && run0 < k) || (open && lane == k - 1));
    const double D = exact ? exact_distance(xq, P.XC + (int64_t)c * d, d, rows_by_16(P.XQ, d) && rows_by_16(P.XC, d)) : 0.0;
    int rank = run0;
    for (int r = 1; __any(lane - r >= run0 || lane + r <= run1); ++r) {
        const double Dl = __shfl(D, lane - r, G), Dr = __shfl(D, lane + r, G);
        const int32_t cl = __shfl(c, lane - r, G), cr = __shfl(c, lane + r, G);
        if (lane - r >= run0 && (Dl < D || (Dl == D && cl < c))) ++rank;
        if (lane + r <= run1 && (Dr < D || (Dr == D && cr < c))) ++rank;
    }
    if (c >= 0 && rank < k) out[(int64_t)q * k + rank] = c;
    if (lane >= cnt && lane < k) out[(int64_t)q * k + lane] = -1;   // fewer than k candidates in the group, or in the slice fewer near enough
    // (of a slice with fewer, a lane's list may have run over all the same: 16-row tiles, lists of 12)
    if (P.shared && lane == 0 && cnt < k && t < __builtin_inff()) flagged[atomicAdd(n_flagged, 1u)] = q;
    if (!open) return;
    // |q'|^2 of the centred query as the filter saw it: the group's lanes add a strided share each (the order is free: the
    // value only enters an inequality with slack)
    double qn = 0.0;
    const float* ctr = P.centre + (int64_t)g * d;
    for (int x = lane; x < d; x += G) {
        const double v = (double)(xq[x] - ctr[x]);
        qn = fma(v, v, qn);
    }
    for (int w = G / 2; w > 0; w >>= 1) qn += __shfl_xor(qn, w, G);
    if (c >= 0 && rank == k - 1 && !(D - qn + eps < (double)t)) flagged[atomicAdd(n_flagged, 1u)] = q;
}

// ---------------------------------------------------------------- stage 3: flagged queries, exactly, against the whole cluster
// exact distances of four rows at once (the chains side by side); rows without a candidate (c < 0) can be read and count for nothing
__device__ __forceinline__ void exact_distances4(const float* __restrict__ x, const float* const (&y)[4], const int32_t (&c)[4], int32_t d, bool by16,
                                                 double (&D)[4]) {
    if (d > 32) {   // long rows keep enough loads in flight by themselves
#pragma unroll
        for (int u = 0; u < 4; ++u) D[u] = c[u] >= 0 ? exact_distance(x, y[u], d, by16) : 0.0;
        return;
    }
    double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int t = 0; t < d; ++t) {
        const double xt = (double)x[t];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double diff = xt - (double)y[u][t];
            a[u] = __dadd_rn(a[u], __dmul_rn(diff, diff));
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) D[u] = a[u];
}

// A team of THREADS lanes, a workgroup or one wavefront of it, per flagged query (or part of its group) at a time.  Every lane
// walks its share of the candidates once, four at a time, and keeps its own k smallest (distance, point) pairs sorted in
// registers (KL >= k slots); the k smallest of all are among those, and k rounds pick them: each lane offers its smallest pair
// above the one picked before, the team takes the smallest offer.
template <int KL, int THREADS>
struct ExactTeam {
    double lD[KL];      // ascending in (distance, point); empty slots: (inf, -1) at the end
    int32_t lP[KL];
    double wD;          // the pair in slot k - 1 (point -1 while the list is not full)
    int32_t wP;

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int x = 0; x < KL; ++x) { lD[x] = __builtin_inf(); lP[x] = -1; }
        wD = __builtin_inf();
        wP = -1;
    }
    __device__ __forceinline__ void insert(double xD, int32_t xP, int32_t k) {
        // slot k - 1 is the list's last used slot: what does not come before it cannot be among this thread's k smallest
        if (!(wP < 0 || xD < wD || (xD == wD && xP < wP))) return;
#pragma unroll
        for (int x = 0; x < KL; ++x) {
            if (x < k) {
                const bool take = xP >= 0 && (lP[x] < 0 || xD < lD[x] || (xD == lD[x] && xP < lP[x]));
                const double oD = lD[x];
                const int32_t oP = lP[x];
                lD[x] = take ? xD : oD;
                lP[x] = take ? xP : oP;
                xD = take ? oD : xD;
                xP = take ? oP : xP;
            }
        }
#pragma unroll
        for (int x = 0; x < KL; ++x)
            if (x == k - 1) { wD = lD[x]; wP = lP[x]; }
    }
    // the candidates at positions c0 .. c1 - 1
    __device__ __forceinline__ void walk(const KnnSets& P, int32_t q, int32_t k, uint32_t c0, uint32_t c1) {
        const int32_t d = P.d;
        const float* xq = P.XQ + (int64_t)q * d;
        const bool by16 = rows_by_16(P.XQ, d) && rows_by_16(P.XC, d);
        const int32_t self = P.self_row ? P.self_row[q] : P.same_set ? q : -1;
        for (uint32_t pos = c0 + threadIdx.x % THREADS; pos < c1; pos += 4 * THREADS) {
            int32_t c[4];
            const float* row[4];
            double D[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = pos + u * THREADS < c1 ? knn_row(P.cmembers, pos + u * THREADS) : -1;
                row[u] = P.XC + (int64_t)(c[u] < 0 ? knn_row(P.cmembers, pos) : c[u]) * d;
            }
            exact_distances4(xq, row, c, d, by16, D);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (c[u] < 0 || c[u] == self) continue;
                insert(D[u] == D[u] ? D[u] : __builtin_inf(), c[u], k);   // no number: as far as can be, so that every candidate has a place in the order
            }
        }
    }
    // put(m, D, P) by the team's first lane for the k smallest in order, point -1 once there are no more
    template <typename Put>
    __device__ __forceinline__ void pick(int32_t k, double* sD, int32_t* sP, const Put& put) {
        const uint32_t tid = threadIdx.x % THREADS;
        double lastD = -1.0;
        int32_t lastP = -1;
        for (int m = 0; m < k; ++m) {
            double bestD = __builtin_inf();
            int32_t bestP = -1;
#pragma unroll
            for (int x = KL - 1; x >= 0; --x) {   // descending, so that the first pair after the last pick is what remains
                const bool after = lP[x] >= 0 && (lD[x] > lastD || (lD[x] == lastD && lP[x] > lastP));
                bestD = after ? lD[x] : bestD;
                bestP = after ? lP[x] : bestP;
            }
            // smallest offer: inside the wavefront, then over the wavefronts' offers
            auto take_smaller = [&](double Do, int32_t Po) {
                const bool take = Po >= 0 && (bestP < 0 || Do < bestD || (Do == bestD && Po < bestP));
                bestD = take ? Do : bestD;
                bestP = take ? Po : bestP;
            };
            for (int w = 32; w > 0; w >>= 1) take_smaller(__shfl_xor(bestD, w, 64), __shfl_xor(bestP, w, 64));
            if (THREADS > 64) {
                if ((tid & 63) == 0) { sD[tid >> 6] = bestD; sP[tid >> 6] = bestP; }
                __syncthreads();
                bestD = __builtin_inf();
                bestP = -1;
                for (int w = 0; w < THREADS / 64; ++w) take_smaller(sD[w], sP[w]);
            }
            lastD = bestD;
            lastP = bestP;
            if (tid == 0) put(m, lastD, lastP);
            if (THREADS > 64) __syncthreads();
            if (lastP < 0) {   // nothing left: the remaining slots stay empty
                if (tid == 0)
                    for (int x = m + 1; x < k; ++x) put(x, lastD, -1);
                break;
            }
        }
    }
};
template <int KL, int THREADS>
__device__ __forceinline__ void exact_query(const KnnSets& P, int32_t q, int32_t k, int32_t* __restrict__ out, double* sD, int32_t* sP) {
    const int32_t r = P.group_of_q ? P.group_of_q[q] : 0;
    ExactTeam<KL, THREADS> team;
    team.clear();
    team.walk(P, q, k, P.cstart[r], P.cstart[r + 1]);
    team.pick(k, sD, sP, [&](int m, double, int32_t c) { out[(int64_t)q * k + m] = c; });
}

// Work space for queries whose groups are cut: pairs of every workgroup, and per query how many of its parts are through (zero)
struct ExactParts { double* D; int32_t* P; uint32_t* done; };   // [grid * k] each, [grid] (one per query, at most half of them used)
constexpr uint32_t kMaxParts = 32;

// The teams take the flagged queries in turn (how many there are is known on the device only).  Usually there are a few dozen: the
// time is one query's chain of memory latencies.  Up to half as many as workgroups: the query's group is cut into parts of at
// least a row for every lane, a workgroup each, and the one that is through last picks from all parts' pairs (100,003 x 768:
// 0.51 ms with a workgroup to a query, now 0.22; 1,000,000 x 128 in 256 clusters: 0.15 to 0.19, now 0.09).  Up to four a
// workgroup: a workgroup each.  From there on (data with far outliers, groups the filter cannot work on) a wavefront each: the k
// rounds then need no barriers and short groups leave fewer lanes without a candidate.  Whole calls, a workgroup each -> a wavefront each: 200,000 x 64 in 64 clusters, k = 15, 62,000 and 145,000
// flagged 29 -> 12.5 and 64 -> 27 ms, 3,100 flagged 2.35 -> 1.6; 20,000 x 768, 7,300 flagged 14.8 -> 7.0; five iterations of
// 300,000 x 128 on 128 centroids, all flagged, 59 -> 14; one cluster of 100,000 x 128, 9,600 flagged 78 -> 81 (both bound by the
// rows' way from the last cache).
template <int KL, int THREADS>
__global__ void __launch_bounds__(THREADS) k_knn_exact(const KnnSets P, const int32_t* __restrict__ flagged, const uint32_t* __restrict__ n_flagged,
                                                       int32_t k, int32_t* __restrict__ out, const ExactParts parts) {
    __shared__ double sD[THREADS / 64];
    __shared__ int32_t sP[THREADS / 64];
    __shared__ uint32_t through;
    constexpr uint32_t kWaves = THREADS / 64;
    const uint32_t count = *n_flagged;
    if (count >= 4u * gridDim.x) {
        for (uint32_t f = blockIdx.x * kWaves + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6); f < count; f += gridDim.x * kWaves)
            exact_query<KL, 64>(P, flagged[f], k, out, sD, sP);
        return;
    }
    if (KL == 1 || 2u * count > gridDim.x) {   // (one neighbour wanted: the candidates are a few hundred centroids)
        for (uint32_t f = blockIdx.x; f < count; f += gridDim.x) {
            exact_query<KL, THREADS>(P, flagged[f], k, out, sD, sP);
            __syncthreads();
        }
        return;
    }
    if (count == 0u) return;
    const uint32_t f = blockIdx.x % count, part = blockIdx.x / count;
    const int32_t q = flagged[f], r = P.group_of_q ? P.group_of_q[q] : 0;
    const uint32_t c0 = P.cstart[r], c1 = P.cstart[r + 1];
    const uint32_t n_parts = max(1u, min(min(kMaxParts, gridDim.x / count), (c1 - c0 + THREADS - 1u) / THREADS));
    if (part >= n_parts) return;
    if (n_parts == 1u) { exact_query<KL, THREADS>(P, q, k, out, sD, sP); return; }
    const uint32_t span = (c1 - c0 + n_parts - 1u) / n_parts, from = min(c1, c0 + part * span);
    ExactTeam<KL, THREADS> team;
    team.clear();
    team.walk(P, q, k, from, min(c1, from + span));
    team.pick(k, sD, sP, [&](int m, double D, int32_t c) { parts.D[(size_t)blockIdx.x * k + m] = D; parts.P[(size_t)blockIdx.x * k + m] = c; });
    if (threadIdx.x == 0) {
        __threadfence();
        through = atomicAdd(&parts.done[f], 1u) + 1u;
    }
    __syncthreads();
    if (through != n_parts) return;
    __threadfence();
    team.clear();
    for (uint32_t x = threadIdx.x; x < n_parts * (uint32_t)k; x += THREADS) {
        const size_t at = ((size_t)(x / (uint32_t)k) * count + f) * k + x % (uint32_t)k;
        if (parts.P[at] >= 0) team.insert(parts.D[at], parts.P[at], k);
    }
    __syncthreads();
    team.pick(k, sD, sP, [&](int m, double, int32_t c) { out[(int64_t)q * k + m] = c; });
}

// One neighbour wanted, queries the filter's bound could not decide: the exact distances of the `width` (4 or 8)
// candidates the filter kept, one lane each; certified as in k_knn_refine.  One group of queries, which are rows; the filter's bits say which of a tile are
// open.  A wavefront takes `tiles` tiles (refine_tiles), queues their open queries in LDS, and then 64 / width of them at a time, each a chain of d
// additions: as many wavefronts as there can be, and the tiles of one as far apart as can be, for open queries lie together where the rows are in
// the order of their classes.
__global__ void __launch_bounds__(256) k_assign_refine(const KnnSets P, const uint32_t* __restrict__ open, int64_t n_tiles, int32_t tile, int32_t tiles,
                                                       const int32_t* __restrict__ cand, const float* __restrict__ tau, int32_t width,
                                                       int32_t* __restrict__ out, int32_t* __restrict__ flagged, uint32_t* __restrict__ n_flagged) {
    __shared__ int32_t queues[4][kRefineTiles * 32];
    int32_t* const queue = queues[threadIdx.x >> 6];
    const uint32_t in_wave = threadIdx.x & 63u, lane = threadIdx.x % (uint32_t)width, per = 64u / (uint32_t)width;
    const int64_t t = (int64_t)in_wave * gridDim.x * 4 + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // this lane's tile
    uint32_t bits = in_wave < (uint32_t)tiles && t < n_tiles ? open[t] : 0u;
    uint32_t incl = (uint32_t)__popc(bits);
    for (int w = 1; w < kRefineTiles; w <<= 1) {
        const uint32_t up = __shfl_up(incl, w, 64);
        if (in_wave >= (uint32_t)w) incl += up;
    }
    uint32_t at = incl - (uint32_t)__popc(bits);
    const uint32_t count = __shfl(incl, kRefineTiles - 1, 64);
    for (; bits; bits &= bits - 1u) queue[at++] = (int32_t)(t * tile) + __ffs((int)bits) - 1;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");   // (the queue is the wavefront's own)
    for (uint32_t y = in_wave / (uint32_t)width; y < count; y += per) {
        const int32_t x = queue[y], q = x, g = 0;
        if (!knn_filter_usable(P.Q.max_bits[g], P.C.max_bits[g])) {
            if (lane == 0u) flagged[atomicAdd(n_flagged, 1u)] = q;
            continue;
        }
        const float* xq = P.XQ + (int64_t)q * P.d;
        const int32_t c = cand[(size_t)x * width + lane];
        double D = c >= 0 ? exact_distance(xq, P.XC + (int64_t)c * P.d, P.d, rows_by_16(P.XQ, P.d) && rows_by_16(P.XC, P.d)) : __builtin_inf();
        int32_t best = c >= 0 ? c : 0x7fffffff;
        double qn = 0.0;
        const float* ctr = P.centre + (int64_t)g * P.d;
        for (int t = (int)lane; t < P.d; t += width) {
            const double v = (double)(xq[t] - ctr[t]);
            qn = fma(v, v, qn);
        }
        for (int w = width / 2; w > 0; w >>= 1) {
            const double oD = __shfl_xor(D, w, 64);
            const int32_t oc = __shfl_xor(best, w, 64);
            qn += __shfl_xor(qn, w, 64);
            if (oD < D || (oD == D && oc < best)) { D = oD; best = oc; }
        }
        if (lane != 0u) continue;
        const bool found = best != 0x7fffffff;
        if (found) out[q] = best;
        const double eps = knn_filter_eps(P.d, fmax((double)__uint_as_float(P.Q.max_bits[g]), (double)__uint_as_float(P.C.max_bits[g])), P.chunk);
        const float t = tau[x];
        if (!found || (t < __builtin_inff() && !(D - qn + eps < (double)t))) flagged[atomicAdd(n_flagged, 1u)] = q;
    }
}

// ---------------------------------------------------------------- Lloyd's iterations (the K-Means index of Section 3.2)
// ---- stable sort of the points by label (the M step adds a cluster's rows in ascending point order)
// Least-significant-digit radix passes of 8 bits over (label, point) pairs.  A workgroup of 256 lanes owns kSortSpan
// consecutive positions of a pass's input: it counts its digits (k_sort_count), an exclusive scan over the counts in
// (digit, workgroup) order gives every workgroup the first output slot of each of its digits (two levels), and the
// scatter (k_sort_scatter) ranks the pairs of a chunk of 256 in input order: inside a wavefront by the lanes below
// with the same digit (eight ballots), across wavefronts by their counts taken in wavefront order, across chunks by a
// running slot per digit.  Equal digits keep their input order in every pass, so equal labels end up in ascending
// point order.
constexpr int kSortSpan = 2048;

// One lane of every workgroup adds what the workgroup counted; the last of them hands the sum to the host.  Count and workgroups share
// a word (sum in the high half), so that one atomic does and nothing has to be fenced (a fence writes the XCD's L2 back: the
// count of a million labels took 11.5 us with one, 5.4 without).
__device__ __forceinline__ void report_changed(uint32_t count, uint32_t workgroups, unsigned long long* __restrict__ changed,
                                               unsigned long long* __restrict__ changed_host, const uint32_t* __restrict__ open_count = nullptr) {
    const unsigned long long before = atomicAdd(changed, ((unsigned long long)count << 32) + 1ull);
    if ((uint32_t)before + 1u == workgroups)
        *(volatile unsigned long long*)changed_host = (before >> 32) + count + (open_count ? (unsigned long long)*open_count << 32 : 0ull);
}

// Which clusters the M step computes: those that a point has entered or left since the step before.  The others' means are what they were, bit for
// bit, for a centroid is its members' sum in ascending order.  The stamp of an iteration stands for "changed", so that nothing has to be cleared
// between two; nullptr: all of them.  In Gaussian mixtures (1,000,000 x 128 in 256 clusters) the share of the points in such clusters goes 0.99, 0.48,
// 0.21, 0.10, 0.07, .. by iteration, in rows without structure it stays 1.  There, ten iterations: partial sums 1.19 -> 0.52 ms, a call 5.49 -> 4.68.
struct ChangedClusters {
    int32_t* stamp_of;
    int32_t stamp, n;
    __device__ __forceinline__ bool has(int32_t j) const { return !stamp_of || stamp_of[j] == stamp; }
    __device__ __forceinline__ void add(int32_t j) const { if (stamp_of[j] != stamp) stamp_of[j] = stamp; }   // (whoever writes it writes the same)
};

constexpr int kMarkLds = 1024;   // clusters up to which a workgroup marks its own in LDS first (straight into the stamps: 130,000 labels of 8 9.6 us, now 7.2)
// With prev it also counts the keys that differ from prev's, and marks their clusters; with changed_host the last workgroup hands the count to the
// host, which waits for it while the sort goes on, and in the high half what the filter has counted (open_count).  Without prev the stamps of
// n_clear clusters are cleared.
__global__ void __launch_bounds__(256) k_sort_count(const int32_t* __restrict__ keys, int64_t n, int shift, uint32_t n_blocks,
                                                    uint32_t* __restrict__ hist, const int32_t* __restrict__ prev,   // hist [256][n_blocks]
                                                    unsigned long long* __restrict__ changed, unsigned long long* __restrict__ changed_host, const uint32_t* __restrict__ open_count,
                                                    ChangedClusters clusters, int32_t n_clear) {
    __shared__ uint32_t h[256], moved, of_cluster[kMarkLds];
    const bool local = clusters.n <= kMarkLds;   // marks of the workgroup's clusters in LDS first
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; !prev && j < n_clear; j += (int64_t)gridDim.x * 256) clusters.stamp_of[j] = 0;
    h[threadIdx.x] = 0u;
    if (threadIdx.x == 0) moved = 0u;
    for (int32_t j = threadIdx.x; prev && local && j < clusters.n; j += 256) of_cluster[j] = 0u;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * kSortSpan;
    constexpr int kPer = kSortSpan / 256;
    int32_t key[kPer], before[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int64_t i = i0 + u * 256 + threadIdx.x;
        key[u] = i < n ? keys[i] : 0;
        before[u] = prev && i < n ? prev[i] : key[u];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (i0 + u * 256 + threadIdx.x < n) atomicAdd(&h[((uint32_t)key[u] >> shift) & 255u], 1u);
        if (prev) {
            const bool other = key[u] != before[u];
            if (other && local) of_cluster[key[u]] = of_cluster[before[u]] = 1u;
            else if (other) { clusters.add(key[u]); clusters.add(before[u]); }
            const unsigned long long differ = __ballot(other);
            if (differ && (threadIdx.x & 63) == 0) atomicAdd(&moved, (uint32_t)__popcll(differ));
        }
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * n_blocks + blockIdx.x] = h[threadIdx.x];
    for (int32_t j = threadIdx.x; prev && local && moved && j < clusters.n; j += 256)
        if (of_cluster[j]) clusters.add(j);
    if (changed_host && threadIdx.x == 0) report_changed(moved, gridDim.x, changed, changed_host, open_count);
}

// Exclusive scan of the m counters in two levels: every workgroup scans a tile of kScanTile consecutive counters in
// place and reports the tile's total (k_sort_scan_tiles); one workgroup scans the totals (k_sort_scan); the scatter adds
// a counter's tile offset when it reads it.
constexpr int kScanTile = 2048;

__global__ void __launch_bounds__(256) k_sort_scan_tiles(uint32_t* __restrict__ hist, uint64_t m, uint32_t* __restrict__ tile_total) {
    __shared__ uint32_t wave_sum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t x0 = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * 8;
    uint32_t v[8];
    uint32_t own = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) { v[u] = x0 + u < m ? hist[x0 + u] : 0u; own += v[u]; }
    uint32_t incl = own;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const uint32_t up = __shfl_up(incl, dlt, 64);
        if (lane >= dlt) incl += up;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - own;
    for (int w = 0; w < wave; ++w) run += wave_sum[w];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if (x0 + u < m) hist[x0 + u] = run;
        run += v[u];
    }
    if (threadIdx.x == 255) tile_total[blockIdx.x] = run;
}

// exclusive scan of m counters in place; one workgroup, every lane a contiguous share
__global__ void __launch_bounds__(1024) k_sort_scan(uint32_t* __restrict__ hist, uint64_t m) {
    __shared__ uint32_t part[1024];
    const uint64_t per = (m + 1023) / 1024;
    const uint64_t a = min(m, (uint64_t)threadIdx.x * per), b = min(m, a + per);
    uint32_t own = 0;
    for (uint64_t x = a; x < b; ++x) own += hist[x];
    part[threadIdx.x] = own;
    __syncthreads();
    for (int dlt = 1; dlt < 1024; dlt <<= 1) {
        const uint32_t v = (int)threadIdx.x >= dlt ? part[threadIdx.x - dlt] : 0u;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    uint32_t run = part[threadIdx.x] - own;
    for (uint64_t x = a; x < b; ++x) { const uint32_t c = hist[x]; hist[x] = run; run += c; }
}

// vals_in == nullptr: the value of position i is i (first pass); lstart: see k_label_starts (a single pass only)
__global__ void __launch_bounds__(256) k_sort_scatter(const int32_t* __restrict__ keys_in, const int32_t* __restrict__ vals_in, int64_t n,
                                                      int shift, uint32_t n_blocks, const uint32_t* __restrict__ first_slot,
                                                      const uint32_t* __restrict__ tile_offset, int32_t* __restrict__ keys_out,
                                                      int32_t* __restrict__ vals_out, int32_t K, uint32_t* __restrict__ lstart) {
    __shared__ uint32_t running[256];       // next output slot of every digit for this workgroup
    __shared__ uint32_t wave_cnt[4][256];   // pairs of the chunk with each digit, per wavefront
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    {
        const size_t x = (size_t)threadIdx.x * n_blocks + blockIdx.x;   // the counters in (digit, workgroup) order
        running[threadIdx.x] = first_slot[x] + tile_offset[x / kScanTile];
        if (lstart && blockIdx.x == 0) {   // the only pass: a digit's first slot is its label's
            if ((int32_t)threadIdx.x < K) lstart[threadIdx.x] = running[threadIdx.x];
            if (threadIdx.x == 0) lstart[K] = (uint32_t)n;
        }
    }
    const int64_t i0 = (int64_t)blockIdx.x * kSortSpan;
    for (int u = 0; u < kSortSpan / 256; ++u) {
#pragma unroll
        for (int w = 0; w < 4; ++w) wave_cnt[w][threadIdx.x] = 0u;
        __syncthreads();
        const int64_t i = i0 + u * 256 + threadIdx.x;
        const bool has = i < n;
        const int32_t key = has ? keys_in[i] : 0;
        const int32_t val = has ? (vals_in ? vals_in[i] : (int32_t)i) : 0;
        const uint32_t dgt = ((uint32_t)key >> shift) & 255u;
        unsigned long long same = __ballot(has);   // lanes of this wavefront that hold a pair with this lane's digit
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const bool set = (dgt >> bit) & 1u;
            const unsigned long long m = __ballot(set);
            same &= set ? m : ~m;
        }
        const uint32_t below = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
        if (has && below == 0u) wave_cnt[wave][dgt] = (uint32_t)__popcll(same);
        __syncthreads();
        if (has) {
            uint32_t pos = running[dgt] + below;
            for (int w = 0; w < wave; ++w) pos += wave_cnt[w][dgt];
            keys_out[pos] = key;
            vals_out[pos] = val;
        }
        __syncthreads();
        running[threadIdx.x] += wave_cnt[0][threadIdx.x] + wave_cnt[1][threadIdx.x] + wave_cnt[2][threadIdx.x] + wave_cnt[3][threadIdx.x];
    }
}

// first position of every label in the sorted labels (lstart[K] = n); never a store outside lstart, whatever the labels hold
__global__ void __launch_bounds__(256) k_label_starts(const int32_t* __restrict__ keys, int64_t n, int32_t K, uint32_t* __restrict__ lstart) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    const int32_t cur = i < n ? min(keys[i], K) : K, prev = i > 0 ? max(keys[i - 1], -1) : -1;
    for (int32_t j = prev + 1; j <= cur; ++j) lstart[j] = (uint32_t)i;
}

// M step: centroid j = float32(sum of its rows / count), the rows added in ascending point order in float64 (ids: the
// points sorted by cluster, ascending inside a cluster); an empty cluster keeps its row.
__device__ __forceinline__ double ordered_column_sum(const float* __restrict__ X, int32_t d, const int32_t* __restrict__ ids, uint32_t r0,
                                                     uint32_t r1, int32_t col) {
    double sum = 0.0;
    uint32_t r = r0;
    if (r + 64 <= r1) {   // batches of 64 rows in flight, the additions in order; the next batch's ids travel with this batch's rows
        int32_t idn[64];
#pragma unroll
        for (int u = 0; u < 64; ++u) idn[u] = ids[r + u];
        for (; r + 64 <= r1; r += 64) {
            float v[64];
#pragma unroll
            for (int u = 0; u < 64; ++u) v[u] = X[(int64_t)idn[u] * d + col];
            if (r + 128 <= r1) {
#pragma unroll
                for (int u = 0; u < 64; ++u) idn[u] = ids[r + 64 + u];
            }
#pragma unroll
            for (int u = 0; u < 64; ++u) sum = __dadd_rn(sum, (double)v[u]);
        }
    }
    for (; r + 8 <= r1; r += 8) {
        int32_t id[8];
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) id[u] = ids[r + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = X[(int64_t)id[u] * d + col];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum = __dadd_rn(sum, (double)v[u]);
    }
    for (; r < r1; ++r) sum = __dadd_rn(sum, (double)X[(int64_t)ids[r] * d + col]);
    return sum;
}

// small clusters: one thread per (cluster, column)
__global__ void __launch_bounds__(256) k_kmeans_update(const float* __restrict__ X, int32_t d, const int32_t* __restrict__ ids,
                                                       const uint32_t* __restrict__ start, int32_t K, ChangedClusters clusters, float* __restrict__ C) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= (int64_t)K * d) return;
    const int32_t j = (int32_t)(x / d), col = (int32_t)(x % d);
    const uint32_t r0 = start[j], r1 = start[j + 1];
    if (r1 == r0 || !clusters.has(j)) return;
    C[x] = (float)(ordered_column_sum(X, d, ids, r0, r1, col) / (double)(r1 - r0));
}

// The M step of a small set in one launch, a workgroup per centroid and 64 columns: it finds the centroid's points among the labels
// itself, in order; four wavefronts bring 64 rows to LDS at a time, one adds them, a column a lane.  With prev it also counts the
// labels that changed; the last workgroup hands the count to the host.  Against the sort, its scans and the sums as launches of their
// own: eight for one (mean_in_one_launch says where that pays).
__global__ void __launch_bounds__(256) k_mean_small(const float* __restrict__ X, int32_t n, int32_t d, const int32_t* __restrict__ labels, const int32_t* __restrict__ prev,
                                                    float* __restrict__ C, unsigned long long* __restrict__ changed, unsigned long long* __restrict__ changed_host) {
    extern __shared__ uint16_t ids[];   // [n] the points of this centroid, ascending
    constexpr int V = 64;               // rows of a stage
    __shared__ float stage[2][V][64];
    __shared__ uint32_t wave_count[4], n_changed;
    const int32_t j = (int32_t)blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int U = 8;                // consecutive labels of a lane
    if (threadIdx.x == 0) n_changed = 0u;
    uint32_t m = 0, moved = 0;
    for (int32_t i0 = 0; i0 < n; i0 += 256 * U) {
        const int32_t first = i0 + (int32_t)threadIdx.x * U;
        uint32_t mine = 0;              // a bit per label that is j
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t i = min(first + u, n - 1);
            const bool is = first + u < n && labels[i] == j;
            mine |= is ? 1u << u : 0u;
            if (prev) moved += is && prev[i] != j ? 1u : 0u;
        }
        uint32_t incl = (uint32_t)__popc(mine);
        const uint32_t own = incl;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const uint32_t up = __shfl_up(incl, dlt, 64);
            if (lane >= dlt) incl += up;
        }
        if (lane == 63) wave_count[wave] = incl;
        __syncthreads();
        uint32_t at = m + incl - own;
        for (int w = 0; w < wave; ++w) at += wave_count[w];
        for (; mine; mine &= mine - 1u) ids[at++] = (uint16_t)(first + __ffs((int)mine) - 1);
        m += wave_count[0] + wave_count[1] + wave_count[2] + wave_count[3];
        __syncthreads();
    }
    if (moved && blockIdx.y == 0) atomicAdd(&n_changed, moved);
    if (m) {
        const int32_t col = (int32_t)blockIdx.y * 64 + lane, c = min(col, d - 1);
        float v[V / 4];                 // rows wave, wave + 4, ... of the next stage
        const auto load = [&](uint32_t r0) {   // rows past the end: the last again, not added
#pragma unroll
            for (int u = 0; u < V / 4; ++u) v[u] = X[(int64_t)ids[min(r0 + 4u * u + (uint32_t)wave, m - 1u)] * d + c];
        };
        load(0u);
        double sum = 0.0;
        for (uint32_t r0 = 0, buf = 0; r0 < m; r0 += V, buf ^= 1u) {
#pragma unroll
            for (int u = 0; u < V / 4; ++u) stage[buf][4 * u + wave][lane] = v[u];
            if (r0 + V < m) load(r0 + V);
            __syncthreads();            // (a stage is written again only after the barrier of the one between)
            if (wave == 0) {
                if (r0 + V <= m) {
#pragma unroll
                    for (int u = 0; u < V; ++u) sum = __dadd_rn(sum, (double)stage[buf][u][lane]);
                } else {
                    for (uint32_t u = 0; r0 + u < m; ++u) sum = __dadd_rn(sum, (double)stage[buf][u][lane]);
                }
            }
        }
        if (wave == 0 && col < d) C[(int64_t)j * d + col] = (float)(sum / (double)m);
    }
    if (!changed_host) return;
    __syncthreads();
    if (threadIdx.x == 0) report_changed(n_changed, gridDim.x * gridDim.y, changed, changed_host);
}

// Large clusters.  A chain of thousands of ordered additions per thread leaves most of the chip idle (a million points in
// 256 clusters: 0.33 ms for 512 MB; in parallel 0.11 ms, the card's copy rate).  The centroid is the sum rounded to float32,
// and the 29 bits less hide the order in nearly every case: every addition errs by at most 2^-53 of its result, so from
// bounds on the partial sums of both orders follows an interval that holds the ordered sum, and if both its ends divide and
// round to the same float32, that is the centroid.  The few columns whose interval straddles a rounding boundary (or is not
// finite) are put on a list and added in order.
//
// k_mean_partials: a workgroup takes `span` positions of the sorted order; the part of span b that lies in cluster j is
// partial number b + j (b + j grows along the order, so the numbers are distinct and below spans + K).
// (mean_span, kmeans_plan.h)
struct MeanPartial { double sum; double magnitude; };

template <int VEC>
__global__ void __launch_bounds__(256) k_mean_partials(const float* __restrict__ X, int64_t n, int32_t d, const int32_t* __restrict__ keys,
                                                       const int32_t* __restrict__ ids, const uint32_t* __restrict__ lstart, int32_t span,
                                                       ChangedClusters clusters, MeanPartial* __restrict__ partial) {
    __shared__ double s_sum[4][64 * VEC], s_mag[4][64 * VEC];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t b0 = blockIdx.x * (uint32_t)span, b1 = (uint32_t)min(n, (int64_t)b0 + span);
    for (uint32_t r0 = b0; r0 < b1;) {
        const int32_t j = __builtin_amdgcn_readfirstlane(keys[r0]);
        const uint32_t r1 = min(b1, (uint32_t)__builtin_amdgcn_readfirstlane((int)lstart[j + 1]));
        if (!clusters.has(j)) { r0 = r1; continue; }
        MeanPartial* out = partial + ((size_t)blockIdx.x + (size_t)j) * d;
        for (int c0 = 0; c0 < d; c0 += 64 * VEC) {
            const int col = c0 + lane * VEC;
            const float* src = X + (col < d ? col : 0);
            double sum[VEC], mag[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) sum[v] = mag[v] = 0.0;
            const auto load = [&](uint32_t r, float (&x)[VEC]) {
                const float* row = src + (int64_t)ids[r] * d;
                if constexpr (VEC == 4) { const float4 t = *(const float4*)row; x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w; }
                else if constexpr (VEC == 2) { const float2 t = *(const float2*)row; x[0] = t.x; x[1] = t.y; }
                else x[0] = *row;
            };
            const auto add = [&](const float (&x)[VEC]) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) { sum[v] += (double)x[v]; mag[v] += fabs((double)x[v]); }
            };
            uint32_t r = r0 + (uint32_t)wave;
            for (; r + 60 < r1; r += 64) {   // sixteen rows of this wavefront in flight
                float x[16][VEC];
#pragma unroll
                for (int u = 0; u < 16; ++u) load(r + 4u * u, x[u]);
#pragma unroll
                for (int u = 0; u < 16; ++u) add(x[u]);
            }
            for (; r < r1; r += 4) {
                float x[VEC];
                load(r, x);
                add(x);
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) { s_sum[wave][lane * VEC + v] = sum[v]; s_mag[wave][lane * VEC + v] = mag[v]; }
            __syncthreads();
            for (int x = threadIdx.x; x < 64 * VEC && c0 + x < d; x += 256)
                out[c0 + x] = {(s_sum[0][x] + s_sum[1][x]) + (s_sum[2][x] + s_sum[3][x]), (s_mag[0][x] + s_mag[1][x]) + (s_mag[2][x] + s_mag[3][x])};
            __syncthreads();
        }
        r0 = r1;
    }
}

// The partials of every (cluster, column); columns whose float32 the order could change go on the list (*n_list of them).
// With P_b the sum of the spans before b, m_b, M_b the rows and magnitudes of span b and u = 2^-53: a partial sum of the
// ordered addition inside span b is at most |P_b| + M_b (+ what the earlier roundings moved, below 2 m u M), so it errs by
// at most u sum_b m_b (|P_b| + M_b + 2 m u M); the parallel sum by u (span / 4 + 4) M inside the spans and u |P_b| at each join.
__global__ void __launch_bounds__(256) k_mean_combine(const MeanPartial* __restrict__ partial, int32_t d, const uint32_t* __restrict__ lstart, int32_t K, int32_t span,
                                                      ChangedClusters clusters, float* __restrict__ C, uint32_t* __restrict__ list, uint32_t* __restrict__ n_list) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= (int64_t)K * d) return;
    const int32_t j = (int32_t)(x / d), col = (int32_t)(x % d);
    const uint32_t r0 = lstart[j], r1 = lstart[j + 1];
    if (r1 == r0 || !clusters.has(j)) return;
    double sum = 0.0, mag = 0.0, ordered = 0.0, joins = 0.0;
    const uint32_t b1 = (r1 - 1) / span;
    for (uint32_t b = r0 / span; b <= b1; b += 8) {
        MeanPartial p[8];   // eight loads in flight
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) p[u] = partial[((size_t)min(b + u, b1) + (size_t)j) * d + col];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u)
            if (b + u <= b1) {
                const uint32_t rows = min(r1, (b + u + 1) * span) - max(r0, (b + u) * span);
                ordered += (double)rows * (fabs(sum) + p[u].magnitude);
                sum += p[u].sum;
                mag += p[u].magnitude;
                joins += fabs(sum);
            }
    }
    const double m = (double)(r1 - r0), err = 0x1p-53 * 1.02 * (ordered + joins + mag * (span / 4 + 4 + 2.0 * m * (m * 0x1p-53)));
    const float lo = (float)((sum - err) / m), hi = (float)((sum + err) / m);
    if (lo == hi && mag < 0x1p1000) C[x] = (float)(sum / m);
    else list[atomicAdd(n_list, 1u)] = (uint32_t)x;
}

// the columns on the list, a workgroup each: the values come into LDS in parallel, one wavefront adds them in order
constexpr int kOrderedChunk = 1024;
__global__ void __launch_bounds__(256) k_mean_ordered(const float* __restrict__ X, int32_t d, const int32_t* __restrict__ ids,
                                                      const uint32_t* __restrict__ lstart, const uint32_t* __restrict__ list,
                                                      const uint32_t* __restrict__ n_list, float* __restrict__ C) {
    __shared__ double v[2][kOrderedChunk];
    const uint32_t count = *n_list;
    for (uint32_t e = blockIdx.x; e < count; e += gridDim.x) {
        const uint32_t x = list[e];
        const int32_t j = (int32_t)(x / (uint32_t)d), col = (int32_t)(x % (uint32_t)d);
        const uint32_t r0 = lstart[j], m = lstart[j + 1] - r0;
        const auto stage = [&](uint32_t c) {   // past the end: +0.0, which changes no sum that started from +0.0
#pragma unroll
            for (int u = 0; u < kOrderedChunk / 256; ++u) {
                const uint32_t r = c * kOrderedChunk + 256u * u + threadIdx.x;
                v[c & 1u][256 * u + threadIdx.x] = r < m ? (double)X[(int64_t)ids[r0 + r] * d + col] : 0.0;
            }
        };
        const uint32_t chunks = (m + kOrderedChunk - 1) / kOrderedChunk;
        stage(0);
        double sum = 0.0;
        for (uint32_t c = 0; c < chunks; ++c) {
            __syncthreads();
            if (threadIdx.x < 64) {
                const double* s = v[c & 1u];
#pragma unroll 16
                for (int t = 0; t < kOrderedChunk; ++t) sum = __dadd_rn(sum, s[t]);
            }
            if (c + 1 < chunks) stage(c + 1);
        }
        __syncthreads();   // (the next column's stage overwrites the chunks)
        if (threadIdx.x == 0) C[x] = (float)(sum / (double)m);
    }
}

// The start from a locality-sensitive hash: bit j of a point = [ sum_t h_{j,t} (x_t - a_{j,t}) > 0 ], a_j the anchor row of
// plane j, the sum over t = 0..d-1 in order with difference, product and running sum each rounded once in float64;
// bucket = floor(code K / 2^b).  One, two or four threads per point, one accumulator per plane each.
//
// Only the sign of the sum counts, so it is taken from sum_t h_t x_t - sum_t h_t a_t with fused multiply-adds (a third of the
// operations) wherever that lies outside both sums' roundings, (d + 4) 2^-53 (sum |h_t| |x_t| + sum |h_t| |a_t|) each at most; a point
// on a plane or nearly so (its anchor) walks its row in the order above.  A wavefront's 64 rows come through LDS kLshCols
// columns at a time: whole lines from memory, where a thread walking its own row took 2.1 ms for a million rows of 128.
// P: planes this instance has accumulators for.
// W: wavefronts of a workgroup that share 64 rows, each with kLshCols columns of every W kLshCols; their sums are added at the end (they stand in any order: the bound is
// for that).
constexpr int kMaxPlanes = 30;
constexpr int kLshCols = 16;
// Of every plane j: normals [d][P] as float64 (0 beyond the b planes), and offset [P][3] = sum h a, sum |h| |a|, sum |h|
template <int P>
__global__ void __launch_bounds__(256) k_lsh_table(const float* __restrict__ X, int32_t d, const float* __restrict__ planes,
                                                   const int32_t* __restrict__ anchors, int32_t b, double* __restrict__ normals,
                                                   double* __restrict__ offset) {
    __shared__ double part[4][3];
    const int j = blockIdx.x;
    double s[3] = {0.0, 0.0, 0.0};
    for (int t = threadIdx.x; t < d; t += 256) {
        const double h = j < b ? (double)planes[(int64_t)j * d + t] : 0.0, a = j < b ? (double)X[(int64_t)anchors[j] * d + t] : 0.0;
        normals[(size_t)t * P + j] = h;
        s[0] = fma(h, a, s[0]);
        s[1] = fma(fabs(h), fabs(a), s[1]);
        s[2] += fabs(h);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        for (int w = 32; w > 0; w >>= 1) s[c] += __shfl_xor(s[c], w, 64);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][c] = s[c];
    }
    __syncthreads();
    if (threadIdx.x < 3) offset[3 * j + threadIdx.x] = part[0][threadIdx.x] + part[1][threadIdx.x] + part[2][threadIdx.x] + part[3][threadIdx.x];
}
// How many share.  A row is a chain of d / 16 loads to one wavefront, which few rows wait for; where the rows fill the chip, adding up a row's P sums costs more than it
// saves, and of up to 16 columns there is nothing to share.  us, 1 / 2 / 4 wavefronts, P = 8: 100,000 rows of 32 11 / 9 / 9, of 64 22 / 14 / 12, of 768 210 / 134 / 112; 300,000 of 17
// 10 / 11 / 15, of 32 15 / 14 / 17, of 256 90 / 70 / 66; 1,000,000 of 16 18 / 24 / 36, of 17 21 / 26 / 38, of 32 34 / 32 / 43, of 128 127 / 91 / 91.  P = 16: 100,000 of 64 23 / 18 / 17, of
// 768 226 / 156 / 149, 300,000 of 17 15 / 18 / 26, of 64 32 / 29 / 32, of 256 121 / 95 / 93, 1,000,000 of 64 70 / 76 / 95, of 128 130 / 128 / 149.  P = 32: 100,000 of 17
// 15 / 18 / 22, of 128 66 / 57 / 51, 300,000 of 64 53 / 51 / 58, of 256 224 / 191 / 175, 1,000,000 of 64 119 / 130 / 172, of 128 296 / 288 / 287.
inline int lsh_shared(int64_t n, int32_t d, int P) {
    const double fill = (double)n * P / (double)(1 << 21);
    const int two = fill <= 1.0 ? kLshCols + 1 : fill <= 4.0 ? 2 * kLshCols : 7 * kLshCols, four = fill <= 0.5 ? 2 * kLshCols + 1 : fill <= 1.0 ? 4 * kLshCols : 10 * kLshCols;
    return d < two ? 1 : d < four ? 2 : 4;
}
template <int P, int W>
__global__ void __launch_bounds__(256) k_lsh_buckets(const float* __restrict__ X, int64_t n, int32_t d, const float* __restrict__ planes,
                                                     const int32_t* __restrict__ anchors, const double* __restrict__ normals,
                                                     const double* __restrict__ offset, int32_t b, int32_t K, int32_t* __restrict__ bucket) {
    constexpr int kSets = 4 / W;
    __shared__ float rows[4][64][kLshCols + 1];
    __shared__ double sums[kSets][W > 1 ? P : 1][64];
    __shared__ float bigs[kSets][64];
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), part = wave % W, set = wave / W;
    const int64_t i0 = ((int64_t)blockIdx.x * kSets + set) * 64, i = i0 + lane;
    const int lr = lane / kLshCols, lc = lane % kLshCols;   // loads: column lc of rows lr + 4 u
    double acc[P];
    float big = 0.f;
#pragma unroll
    for (int j = 0; j < P; ++j) acc[j] = 0.0;
    float next[kLshCols];
    const auto load = [&](int t0) {
#pragma unroll
        for (int u = 0; u < kLshCols; ++u) {
            const int64_t r = i0 + lr + (64 / kLshCols) * u;
            next[u] = r < n && t0 + lc < d ? X[r * d + t0 + lc] : 0.f;
        }
    };
    load(part * kLshCols);
    for (int t0 = part * kLshCols; t0 < d; t0 += W * kLshCols) {
        const int cols = min(kLshCols, d - t0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");   // (the rows are the wavefront's own)
#pragma unroll
        for (int u = 0; u < kLshCols; ++u) rows[wave][lr + (64 / kLshCols) * u][lc] = next[u];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        if (t0 + W * kLshCols < d) load(t0 + W * kLshCols);
#pragma unroll 2
        for (int t = 0; t < cols; ++t) {
            const float x = rows[wave][lane][t];
            const double* h = normals + (size_t)(t0 + t) * P;
            big = fmaxf(big, fabsf(x));
#pragma unroll
            for (int j = 0; j < P; ++j) acc[j] = fma(h[j], (double)x, acc[j]);
        }
    }
    if constexpr (W > 1) {
        for (int w = W - 1; w > 0; --w) {   // one wavefront after the other, the first one last
            if (part == w) {
#pragma unroll
                for (int j = 0; j < P; ++j) sums[set][j][lane] = w == W - 1 ? acc[j] : sums[set][j][lane] + acc[j];
                bigs[set][lane] = w == W - 1 ? big : fmaxf(bigs[set][lane], big);
            }
            __syncthreads();
        }
        if (part > 0) return;
#pragma unroll
        for (int j = 0; j < P; ++j) acc[j] += sums[set][j][lane];
        big = fmaxf(big, bigs[set][lane]);
    }
    if (i >= n) return;
    uint64_t code = 0;
    uint32_t open = 0;
#pragma unroll
    for (int j = 0; j < P; ++j)
        if (j < b) {
            const double v = acc[j] - offset[3 * j], bound = (double)(4 * d + 32) * 0x1p-53 * (offset[3 * j + 1] + offset[3 * j + 2] * (double)big);
            if (v > bound) code |= (uint64_t)1 << j;
            else if (!(v < -bound)) open |= 1u << j;
        }
    for (; open; open &= open - 1u) {
        const int j = __ffs((int)open) - 1;
        const float *h = planes + (int64_t)j * d, *a = X + (int64_t)anchors[j] * d, *x = X + i * d;
        double sum = 0.0;
        for (int t = 0; t < d; ++t) sum = __dadd_rn(sum, __dmul_rn((double)h[t], __dsub_rn((double)x[t], (double)a[t])));
        if (sum > 0.0) code |= (uint64_t)1 << j;
    }
    bucket[i] = (int32_t)((code * (uint64_t)K) >> b);
}

// Anchors the caller did not draw: plane j goes through the median of a strided sample along its normal.  The sample is the
// m = min(kLshSample, n) points floor(s n / m); projection = sum_t h_{j,t} x_t over t = 0..d-1 in order (product and
// running sum each rounded once in float64); the anchor is the sample point of rank floor(m / 2) in ascending
// (projection, point).  A wavefront takes 64 of the projections of a plane (k_lsh_projections), a workgroup per plane the median, from a
// bitonic sort.  (One workgroup per plane for both, every thread counting its rank among 1,024: 59 us at 128 columns and 136 at
// 768; now 23 and 39.)
constexpr int kLshSample = 1024;
__global__ void __launch_bounds__(64) k_lsh_projections(const float* __restrict__ X, int64_t n, int32_t d, const float* __restrict__ planes, double* __restrict__ proj) {
    const int j = blockIdx.x, s = (int)blockIdx.y * 64 + (int)threadIdx.x;
    const int m = (int)min((int64_t)kLshSample, n);
    const float* h = planes + (int64_t)j * d;
    const float* x = X + (((int64_t)min(s, m - 1) * n) / m) * d;
    double p = 0.0;
    int t = 0;
    if (rows_by_16(X, d)) {
        for (; t + 32 <= d; t += 32) {   // eight 16-byte loads in flight, added one by one in order
            float4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *(const float4*)(x + t + 4 * u);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                p = __dadd_rn(p, __dmul_rn((double)h[t + 4 * u], (double)v[u].x));
                p = __dadd_rn(p, __dmul_rn((double)h[t + 4 * u + 1], (double)v[u].y));
                p = __dadd_rn(p, __dmul_rn((double)h[t + 4 * u + 2], (double)v[u].z));
                p = __dadd_rn(p, __dmul_rn((double)h[t + 4 * u + 3], (double)v[u].w));
            }
        }
    }
    for (; t + 16 <= d; t += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = x[t + u];
#pragma unroll
        for (int u = 0; u < 16; ++u) p = __dadd_rn(p, __dmul_rn((double)h[t + u], (double)v[u]));
    }
    for (; t < d; ++t) p = __dadd_rn(p, __dmul_rn((double)h[t], (double)x[t]));
    if (!(p == p)) p = __builtin_inf();   // no number: last in the order, so that one point has the median's rank
    proj[(size_t)j * kLshSample + s] = s < m ? p : __builtin_inf();
}

__global__ void __launch_bounds__(kLshSample) k_lsh_median_anchors(const double* __restrict__ proj, int64_t n, int32_t* __restrict__ anchors) {
    __shared__ double sproj[kLshSample];
    __shared__ uint16_t sidx[kLshSample];
    const int j = blockIdx.x, s = threadIdx.x;
    const int m = (int)min((int64_t)kLshSample, n);
    sproj[s] = proj[(size_t)j * kLshSample + s];
    // ascending in (projection, sample); sample points are in ascending index order, the places past them come last
    sidx[s] = (uint16_t)s;
    for (int size = 2; size <= kLshSample; size <<= 1)
        for (int dist = size >> 1; dist > 0; dist >>= 1) {
            __syncthreads();
            const int a = 2 * s - (s & (dist - 1)), b = a + dist;   // pair number s of this step
            if (s < kLshSample / 2) {
                const bool up = (a & size) == 0, after = sproj[a] > sproj[b] || (sproj[a] == sproj[b] && sidx[a] > sidx[b]);
                if (after == up) {
                    const double t = sproj[a]; sproj[a] = sproj[b]; sproj[b] = t;
                    const uint16_t u = sidx[a]; sidx[a] = sidx[b]; sidx[b] = u;
                }
            }
        }
    __syncthreads();
    if (s == 0) anchors[j] = (int32_t)(((int64_t)sidx[m / 2] * n) / m);
}

// centroid j starts as the data point floor(j n / K): what an empty bucket keeps
__global__ void __launch_bounds__(256) k_lsh_fallback(const float* __restrict__ X, int64_t n, int32_t d, int32_t K, float* __restrict__ C) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= (int64_t)K * d) return;
    const int64_t j = x / d;
    C[x] = X[((j * n) / K) * d + x % d];
}

// sum over the points of the distance to their centroid, in float64, added in no particular order: sixteen lanes a row, four rows of theirs in
// flight.  Bound by the read of the rows: 1,000,000 x 128 102 us.  The workgroups add to one word, 10 ns each: sixteen wavefronts to a workgroup, few of them
// (2,048 of four: 130,000 x 16 29 us, now 10).
constexpr int kInertiaGrid = 512, kInertiaRows = 256;   // workgroups at most, rows of one at a time
__global__ void __launch_bounds__(1024) k_kmeans_inertia(const float* __restrict__ X, const float* __restrict__ C, int32_t d,
                                                        const int32_t* __restrict__ labels, int64_t n, double* __restrict__ out) {
    __shared__ double wave_sum[16];
    const int part = threadIdx.x % 16;
    const bool vec = rows_by_16(X, d) && rows_by_16(C, d);
    double sum = 0.0;
    const auto add = [&](float a, float b) { const double e = (double)a - (double)b; sum = fma(e, e, sum); };
    for (int64_t i0 = (int64_t)blockIdx.x * kInertiaRows + threadIdx.x / 16; i0 < n; i0 += (int64_t)gridDim.x * kInertiaRows) {
        const float *x[4], *c[4];
        bool in[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + 64 * u;
            in[u] = i < n;
            x[u] = X + (in[u] ? i : i0) * d;
            c[u] = C + (int64_t)labels[in[u] ? i : i0] * d;
        }
        if (vec) {
            for (int t = 4 * part; t < d; t += 64) {
                float4 a[4], b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) { a[u] = *(const float4*)(x[u] + t); b[u] = *(const float4*)(c[u] + t); }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (in[u]) { add(a[u].x, b[u].x); add(a[u].y, b[u].y); add(a[u].z, b[u].z); add(a[u].w, b[u].w); }
            }
        } else {
            for (int t = part; t < d; t += 16) {
                float a[4], b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) { a[u] = x[u][t]; b[u] = c[u][t]; }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (in[u]) add(a[u], b[u]);
            }
        }
    }
    for (int w = 32; w > 0; w >>= 1) sum += __shfl_xor(sum, w, 64);
    if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    sum = threadIdx.x < 16 ? wave_sum[threadIdx.x] : 0.0;
    for (int w = 8; w > 0; w >>= 1) sum += __shfl_xor(sum, w, 64);
    if (threadIdx.x == 0) atomicAdd(out, sum);
}

}  // namespace nomad_knn
