// Device code of the two quality measures of Section 4: neighbourhood preservation (the overlap of exact
// k-neighbourhoods in the data space and in the projection; the neighbourhoods come from the nearest-neighbour kernels
// of knn_kernels.h) and random triplet accuracy (the fraction of random triplets whose two distances from the anchor
// are ordered alike in both spaces).  Distances are the float64 definition of knn_kernels.h (t = 0..d-1 in order), so
// every decision, and with it every count, is exact.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "knn_kernels.h"
#include "philox.h"
#include "rows.h"

namespace nomad_metrics {

constexpr uint32_t kTripletStream = 0x54524950u;   // third counter word of the triplet generator

// out[p] = X[rows[p % period]] (rows == nullptr: row p % period) for p < m: the listed rows, repeated every `period`;
// bad is set where a row lies outside [0, n)
__global__ void __launch_bounds__(256) k_gather_rows(const float* __restrict__ X, int64_t n, int32_t d, const int32_t* __restrict__ rows,
                                                     int64_t period, int64_t m, float* __restrict__ out, int* __restrict__ bad) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= m * d) return;
    const int64_t p = x / d;
    const int32_t t = (int32_t)(x % d);
    const int64_t r = rows ? rows[p % period] : p % period;
    if (r < 0 || r >= n) { *bad = 1; out[x] = 0.f; return; }
    out[x] = X[r * d + t];
}

// block[p] = p / period (may be nullptr); tiled[p] = rows[p % period] (rows == nullptr: p % period) (may be nullptr)
__global__ void __launch_bounds__(256) k_periodic_ids(const int32_t* __restrict__ rows, int64_t period, int64_t m, int32_t* __restrict__ block,
                                                      int32_t* __restrict__ tiled) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= m) return;
    if (block) block[p] = (int32_t)(p / period);
    if (tiled) tiled[p] = rows ? rows[p % period] : (int32_t)(p % period);
}

// The candidate set was cut into `slices` parts and query r has the k nearest of each part in
// part_nbrs[(g * m + r) * k ..]: the k nearest overall are the k smallest (distance, index) among those slices * k <= 256
// candidates.  One workgroup per query, one thread per candidate, rank by counting.
__global__ void __launch_bounds__(256) k_merge_slices(const float* __restrict__ AQ, const float* __restrict__ A, int32_t d,
                                                      const int32_t* __restrict__ part_nbrs, int32_t slices, int64_t m, int32_t k,
                                                      int32_t* __restrict__ out) {
    __shared__ double sD[256];
    __shared__ int32_t sC[256];
    const int64_t r = blockIdx.x;
    const int t = threadIdx.x, total = slices * k;
    int32_t c = -1;
    double D = __builtin_inf();
    if (t < total) {
        c = part_nbrs[((int64_t)(t / k) * m + r) * k + t % k];
        if (c >= 0) D = nomad_knn::exact_distance(AQ + r * d, A + (int64_t)c * d, d, rows_by_16(AQ, d) && rows_by_16(A, d));
        if (!(D == D)) D = __builtin_inf();   // no number: as in the slices' own order
    }
    sD[t] = D;
    sC[t] = c;
    __syncthreads();
    int rank = 0, found = 0;
    for (int o = 0; o < total; ++o) {
        const int32_t co = sC[o];
        if (co < 0) continue;
        ++found;
        const double Do = sD[o];
        if (Do < D || (Do == D && co < c)) ++rank;
    }
    if (c >= 0 && rank < k) out[r * k + rank] = c;
    if (t >= found && t < k) out[r * k + t] = -1;   // fewer than k candidates in all
}

// ---- nearest neighbours in the plane
// In two dimensions the nearest neighbours of a point are in the cells around it: the points are counted into a square
// grid of about kCellPoints points a cell, row by row, so that the cells of one row of a square are one contiguous range.  A
// wavefront takes a query: the smallest square of cells that holds more than k points, their exact distances, the k
// smallest; if a point outside the square could still be nearer, the square that reaches as far as the k-th distance.
// A million points and 10,000 queries: 0.2 ms, where comparing every query with every point took 12 ms on the matrix cores
// and left most queries to the exact path (neighbour distances in the plane are 1e-5 of its squared extent).
// The grid follows the bounding box: a few far points put nearly all others into one cell, and every query reads them all.
// Same sizes with three points 10,000 deviations out: 20 ms (the matrix cores and the exact path: 31), with Cauchy
// coordinates 24 (209), with half of the points in a ten-thousandth of the extent 12 (99).
constexpr int kCellPoints = 6;
constexpr int kMaxGrid = 2048;      // cells per side

// bounding box as (min x, min y, max x, max y) of ordered bit patterns; box must start at (max, max, 0, 0)
__device__ __forceinline__ uint32_t ordered_bits(float v) {
    const uint32_t b = __float_as_uint(v);
    return b & 0x80000000u ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float from_ordered(uint32_t b) { return __uint_as_float(b & 0x80000000u ? b ^ 0x80000000u : ~b); }

__global__ void k_plane_box_clear(uint32_t* __restrict__ box) {
    if (threadIdx.x < 4) box[threadIdx.x] = threadIdx.x < 2 ? 0xFFFFFFFFu : 0u;
}
__global__ void __launch_bounds__(256) k_plane_box(const float* __restrict__ Y, int64_t n, uint32_t* __restrict__ box) {
    uint32_t lx = 0xFFFFFFFFu, ly = 0xFFFFFFFFu, hx = 0u, hy = 0u;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const float2 y = pair_at(Y, i);
        const uint32_t x0 = ordered_bits(y.x), y0 = ordered_bits(y.y);
        lx = min(lx, x0); hx = max(hx, x0);
        ly = min(ly, y0); hy = max(hy, y0);
    }
    for (int w = 32; w > 0; w >>= 1) {
        lx = min(lx, (uint32_t)__shfl_xor((int)lx, w, 64)); hx = max(hx, (uint32_t)__shfl_xor((int)hx, w, 64));
        ly = min(ly, (uint32_t)__shfl_xor((int)ly, w, 64)); hy = max(hy, (uint32_t)__shfl_xor((int)hy, w, 64));
    }
    __shared__ uint32_t waves[4][4];   // of a wavefront: the box; one set of atomics a workgroup (one a wavefront: 98 us for a million points, now 16)
    if ((threadIdx.x & 63) == 0) {
        uint32_t* const w = waves[threadIdx.x >> 6];
        w[0] = lx; w[1] = ly; w[2] = hx; w[3] = hy;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int c = threadIdx.x;
        uint32_t v = waves[0][c];
        for (int w = 1; w < 4; ++w) v = c < 2 ? min(v, waves[w][c]) : max(v, waves[w][c]);
        if (c < 2) { if (v < box[c]) atomicMin(&box[c], v); }     // (the box only grows: a stale read costs an atomic, not the result)
        else if (v > box[c]) atomicMax(&box[c], v);
    }
}

struct PlaneGrid { float x0, y0, inv; double width; };   // cell of x: floor((x - x0) inv), clamped; square cells
__device__ __forceinline__ PlaneGrid plane_grid(const uint32_t* __restrict__ box, int32_t G) {
    PlaneGrid p;
    p.x0 = from_ordered(box[0]);
    p.y0 = from_ordered(box[1]);
    const float side = fmaxf(from_ordered(box[2]) - p.x0, from_ordered(box[3]) - p.y0);
    p.inv = side > 0.f ? (float)G / side : 0.f;
    if (!(p.inv < 3.0e38f)) p.inv = 0.f;                  // an extent too small to divide by: one cell
    p.width = p.inv > 0.f ? 1.0 / (double)p.inv : __builtin_inf();
    return p;
}
__device__ __forceinline__ int plane_cell(float x, float x0, float inv, int32_t G) {
    const float t = (x - x0) * inv;
    return t >= 1.f ? (int)fminf(t, (float)(G - 1)) : 0;   // monotone in x; what is no number goes to cell 0
}

// cell of every point and the number of points per cell
__global__ void __launch_bounds__(256) k_plane_count(const float* __restrict__ Y, int64_t n, const uint32_t* __restrict__ box, int32_t G,
                                                     uint32_t* __restrict__ counts, uint32_t* __restrict__ rank) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const PlaneGrid p = plane_grid(box, G);
    const float2 y = pair_at(Y, i);
    rank[i] = atomicAdd(&counts[plane_cell(y.y, p.y0, p.inv, G) * G + plane_cell(y.x, p.x0, p.inv, G)], 1u);
}
// start: exclusive scan of the counts in two levels (tile_offset per kScanTile cells)
__global__ void __launch_bounds__(256) k_plane_place(const float* __restrict__ Y, int64_t n, const uint32_t* __restrict__ box, int32_t G,
                                                     const uint32_t* __restrict__ start, const uint32_t* __restrict__ tile_offset,
                                                     const uint32_t* __restrict__ rank, float2* __restrict__ pos, int32_t* __restrict__ id) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const PlaneGrid p = plane_grid(box, G);
    const float2 y = pair_at(Y, i);
    const uint32_t c = (uint32_t)(plane_cell(y.y, p.y0, p.inv, G) * G + plane_cell(y.x, p.x0, p.inv, G));
    const uint32_t at = start[c] + tile_offset[c / nomad_knn::kScanTile] + rank[i];
    pos[at] = y;
    id[at] = (int32_t)i;
}

constexpr int kPlaneBuffer = 320;    // candidates a wavefront holds before it reduces them to the k smallest
__global__ void __launch_bounds__(256) k_plane_neighbours(const float* __restrict__ Y, int64_t n, const int32_t* __restrict__ queries, int64_t m,
                                                          int32_t k, const uint32_t* __restrict__ box, int32_t G, const uint32_t* __restrict__ start,
                                                          const uint32_t* __restrict__ tile_offset, const float2* __restrict__ pos,
                                                          const int32_t* __restrict__ id, int32_t* __restrict__ out,
                                                          unsigned long long* __restrict__ bad) {
    __shared__ double sD[4][kPlaneBuffer];
    __shared__ int32_t sI[4][kPlaneBuffer];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r = (int64_t)blockIdx.x * 4 + wave;
    if (r >= m) return;
    const int32_t q = queries ? queries[r] : (int32_t)r;
    if (q < 0 || q >= n) { *bad = 1ull; return; }
    double* bD = sD[wave];
    int32_t* bI = sI[wave];
    const PlaneGrid g = plane_grid(box, G);
    const float2 y = pair_at(Y, q);
    const int cx = plane_cell(y.x, g.x0, g.inv, G), cy = plane_cell(y.y, g.y0, g.inv, G);
    const uint32_t cells = (uint32_t)(G * G);
    auto cell_begin = [&](uint32_t c) { return c < cells ? start[c] + tile_offset[c / nomad_knn::kScanTile] : (uint32_t)n; };
    auto row_range = [&](int row, int rad, uint32_t& a, uint32_t& b) {
        a = cell_begin((uint32_t)(row * G + max(0, cx - rad)));
        b = cell_begin((uint32_t)(row * G + min(G - 1, cx + rad)) + 1u);
    };
    auto wave_fence = []() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // the smallest square with more than k points (the query is one of them)
    int rad = 1;
    for (;; ++rad) {
        uint32_t held = 0;
        for (int row = max(0, cy - rad) + lane; row <= min(G - 1, cy + rad); row += 64) {
            uint32_t a, b;
            row_range(row, rad, a, b);
            held += b - a;
        }
        for (int w = 32; w > 0; w >>= 1) held += (uint32_t)__shfl_xor((int)held, w, 64);
        if (held > (uint32_t)k || (cx - rad <= 0 && cy - rad <= 0 && cx + rad >= G - 1 && cy + rad >= G - 1)) break;
    }
    double limit = __builtin_inf();      // candidates beyond it are not among the k nearest
    int cnt = 0;
    auto reduce = [&]() {                // the k smallest (distance, id) of the buffer, in order; limit follows
        constexpr int kOwn = (kPlaneBuffer + 63) / 64;
        double D[kOwn];
        int32_t I[kOwn];
        int rank[kOwn];
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
            const int e = lane + 64 * u;
            D[u] = e < cnt ? bD[e] : __builtin_inf();
            I[u] = e < cnt ? bI[e] : 0x7fffffff;
            rank[u] = 0;
        }
        for (int o = 0; o < cnt; ++o) {
            const double Do = bD[o];
            const int32_t Io = bI[o];
#pragma unroll
            for (int u = 0; u < kOwn; ++u) rank[u] += (Do < D[u] || (Do == D[u] && Io < I[u])) ? 1 : 0;
        }
        wave_fence();
#pragma unroll
        for (int u = 0; u < kOwn; ++u)
            if (lane + 64 * u < cnt && rank[u] < k) { bD[rank[u]] = D[u]; bI[rank[u]] = I[u]; }
        wave_fence();
        cnt = min(cnt, k);
        if (cnt == k) limit = bD[k - 1];
    };
    while (true) {
        cnt = 0;
        for (int row = max(0, cy - rad); row <= min(G - 1, cy + rad); ++row) {
            uint32_t a, b;
            row_range(row, rad, a, b);
            for (uint32_t p0 = a; p0 < b; p0 += 64) {
                const uint32_t p = p0 + (uint32_t)lane;
                bool take = p < b;
                double D = 0.0;
                int32_t c = 0;
                if (take) {
                    const float2 v = pos[p];
                    c = id[p];
                    // the exact distance: coordinate by coordinate, difference, product and sum each rounded once
                    const double ex = (double)y.x - (double)v.x, ey = (double)y.y - (double)v.y;
                    D = __dadd_rn(__dmul_rn(ex, ex), __dmul_rn(ey, ey));
                    take = c != q && D <= limit;
                }
                const unsigned long long mask = __ballot(take);
                if (take) {
                    const int e = cnt + (int)__popcll(mask & ((1ull << lane) - 1ull));
                    bD[e] = D;
                    bI[e] = c;
                }
                cnt += (int)__popcll(mask);
                wave_fence();
                if (cnt > kPlaneBuffer - 64) reduce();
            }
        }
        reduce();
        // a point outside the square is at least as far as the square's nearest open side (a hundredth of a cell of slack
        // covers the rounding of the cell numbers)
        double open = __builtin_inf();
        if (cx - rad > 0) open = fmin(open, (double)y.x - ((double)g.x0 + ((double)(cx - rad) + 0.01) * g.width));
        if (cy - rad > 0) open = fmin(open, (double)y.y - ((double)g.y0 + ((double)(cy - rad) + 0.01) * g.width));
        if (cx + rad < G - 1) open = fmin(open, (double)g.x0 + ((double)(cx + rad + 1) - 0.01) * g.width - (double)y.x);
        if (cy + rad < G - 1) open = fmin(open, (double)g.y0 + ((double)(cy + rad + 1) - 0.01) * g.width - (double)y.y);
        if (open == __builtin_inf() || (cnt == k && limit < (open > 0.0 ? open * open : 0.0) * (1.0 - 1e-12))) break;
        // reach as far as the k-th distance (or, short of k points, twice as far as before)
        const double reach = cnt == k ? sqrt(limit) / g.width + 1.1 : 2.0 * rad;
        rad = max(rad + 1, reach < (double)G ? (int)reach + 1 : G);
    }
    if (lane < k) out[r * k + lane] = lane < cnt ? bI[lane] : -1;
}

// common members of the two neighbour lists of every query (-1 = empty slot), summed
__global__ void __launch_bounds__(256) k_overlap(const int32_t* __restrict__ a, const int32_t* __restrict__ b, int32_t k, int64_t m,
                                                 unsigned long long* __restrict__ hits) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int found = 0;
    if (p < m) {
        for (int x = 0; x < k; ++x) {
            const int32_t v = a[p * k + x];
            if (v < 0) continue;
            for (int y = 0; y < k; ++y) found += b[p * k + y] == v;
        }
    }
    for (int w = 32; w > 0; w >>= 1) found += __shfl_xor(found, w, 64);
    if ((threadIdx.x & 63) == 0 && found) atomicAdd(hits, (unsigned long long)found);
}

// squared distances from row a to rows b and c: difference, product and running sum each rounded once in float64,
// t = 0..d-1 in order (two independent chains)
__device__ __forceinline__ void anchor_distances(const float* __restrict__ a, const float* __restrict__ b, const float* __restrict__ c,
                                                 int32_t d, bool by16, double& Dab, double& Dac) {
    double s1 = 0.0, s2 = 0.0;
    int t = 0;
    if (by16) {
        for (; t + 8 <= d; t += 8) {   // six loads in flight
            const float4 a0 = *(const float4*)(a + t), a1 = *(const float4*)(a + t + 4);
            const float4 b0 = *(const float4*)(b + t), b1 = *(const float4*)(b + t + 4);
            const float4 c0 = *(const float4*)(c + t), c1 = *(const float4*)(c + t + 4);
            const float av[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
            const float bv[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
            const float cv[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const double e1 = (double)av[u] - (double)bv[u], e2 = (double)av[u] - (double)cv[u];
                s1 = __dadd_rn(s1, __dmul_rn(e1, e1));
                s2 = __dadd_rn(s2, __dmul_rn(e2, e2));
            }
        }
    }
    for (; t < d; ++t) {
        const double e1 = (double)a[t] - (double)b[t], e2 = (double)a[t] - (double)c[t];
        s1 = __dadd_rn(s1, __dmul_rn(e1, e1));
        s2 = __dadd_rn(s2, __dmul_rn(e2, e2));
    }
    Dab = s1;
    Dac = s2;
}

// The same with the wavefront's rows read together, for rows of 128 bytes and more: eight lanes take 128 consecutive bytes of one
// of the 192 rows, 24 such loads a round for the next 32 columns while the present ones go through LDS to the lanes that own
// them.  A lane that reads its own three rows 16 bytes at a time finds their lines gone from the first cache when it comes to
// their next bytes: a million triplets of 1,000,000 x 128 took 0.76 ms, now 0.29; the 1.2e7 lines alone are 0.21 at the rate
// of gathers from memory.  Every lane of the wavefront takes part; i, j, k are rows of X.
constexpr int32_t kStagedColumns = 32, kStagedPitch = kStagedColumns / 4 + 1;   // (a pitch of nine pieces: no bank conflicts)
struct StagedRows { float4 piece[3 * 64][kStagedPitch]; };
__device__ __forceinline__ void staged_distances(StagedRows& lds, const float* __restrict__ X, int32_t d, uint32_t i, uint32_t j, uint32_t k, double& Dij, double& Dik) {
    const int lane = threadIdx.x & 63, sub = lane & 7, owner = lane >> 3;
    const bool by16 = rows_by_16(X, d);
    uint32_t row[24];
#pragma unroll
    for (int u = 0; u < 24; ++u) row[u] = (uint32_t)__shfl((int)(u < 8 ? i : u < 16 ? j : k), (u & 7) * 8 + owner, 64);
    float4 next[24];
    const auto fetch = [&](int32_t c0) {
        const int32_t col = c0 + 4 * sub;
        if (by16) {
#pragma unroll
            for (int u = 0; u < 24; ++u) next[u] = col < d ? *(const float4*)(X + (int64_t)row[u] * d + col) : make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
#pragma unroll
            for (int u = 0; u < 24; ++u) {
                const float* x = X + (int64_t)row[u] * d;
                next[u] = make_float4(col < d ? x[col] : 0.f, col + 1 < d ? x[col + 1] : 0.f, col + 2 < d ? x[col + 2] : 0.f, col + 3 < d ? x[col + 3] : 0.f);
            }
        }
    };
    double s1 = 0.0, s2 = 0.0;
    fetch(0);
    for (int32_t c0 = 0; c0 < d; c0 += kStagedColumns) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 24; ++u) lds.piece[(u >> 3) * 64 + (u & 7) * 8 + owner][sub] = next[u];
        __syncthreads();
        if (c0 + kStagedColumns < d) fetch(c0 + kStagedColumns);
        // (columns past the last one are zeros in all three rows: they add +0 to sums that are not below it)
#pragma unroll
        for (int p = 0; p < kStagedColumns / 4; ++p) {
            const float4 a = lds.piece[lane][p], b = lds.piece[64 + lane][p], c = lds.piece[128 + lane][p];
            const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w}, cv[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double e1 = (double)av[u] - (double)bv[u], e2 = (double)av[u] - (double)cv[u];
                s1 = __dadd_rn(s1, __dmul_rn(e1, e1));
                s2 = __dadd_rn(s2, __dmul_rn(e2, e2));
            }
        }
    }
    Dij = s1;
    Dik = s2;
}

// Triplet number t (one per thread): anchor i and two other points j, k, all distinct and uniform, from the words of
// Philox(counter = (lo32 t, hi32 t, stream, 0), key = seed) by multiply-high range reduction over n, n - 1 and n - 2
// values, stepping over the points already taken.  It agrees when [D_X(i,j) < D_X(i,k)] == [D_Y(i,j) < D_Y(i,k)].
// A launch covers the triplets t_begin .. t_end-1 and adds its count to *agree.  Workgroups of one wavefront.
template <bool STAGED>
__global__ void __launch_bounds__(64) k_triplets(const float* __restrict__ X, int32_t d, const float* __restrict__ Y, int32_t d_low,
                                                 uint32_t n, int64_t t_begin, int64_t t_end, uint32_t key0, uint32_t key1,
                                                 unsigned long long* __restrict__ agree) {
    __shared__ uint4 space[STAGED ? sizeof(StagedRows) / 16 : 1];
    const int64_t t = t_begin + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // (lanes past the end draw a triplet too, and do not count it)
    uint32_t w[4];
    philox4x32_10((uint32_t)t, (uint32_t)((uint64_t)t >> 32), kTripletStream, 0u, key0, key1, w);
    const uint32_t i = __umulhi(w[0], n);
    uint32_t j = __umulhi(w[1], n - 1u);
    j += j >= i;
    uint32_t k = __umulhi(w[2], n - 2u);
    const uint32_t lo = min(i, j), hi = max(i, j);
    k += k >= lo;
    k += k >= hi;
    double hij, hik, lij, lik;
    anchor_distances(Y + (int64_t)i * d_low, Y + (int64_t)j * d_low, Y + (int64_t)k * d_low, d_low, rows_by_16(Y, d_low), lij, lik);
    if (STAGED) staged_distances(*(StagedRows*)space, X, d, i, j, k, hij, hik);
    else anchor_distances(X + (int64_t)i * d, X + (int64_t)j * d, X + (int64_t)k * d, d, rows_by_16(X, d), hij, hik);
    const bool same = t < t_end && (hij < hik) == (lij < lik);
    const unsigned long long m = __ballot(same);
    if (threadIdx.x == 0 && m) atomicAdd(agree, (unsigned long long)__popcll(m));
}

// *p = v (one lane): clears a counter without a memset node, so that a caller may record the call into a HIP graph
__global__ void k_store_u64(unsigned long long* __restrict__ p, unsigned long long v) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *p = v;
}

}  // namespace nomad_metrics
