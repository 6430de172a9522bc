// Device kernels of the mean-field sums (K2) by interpolation, for problems of many heads and cells.
//
// A(theta) = sum_r p_r q(theta, mu_r) and B(theta) = sum_r p_r q^2 (theta - mu_r) over all cells are smooth functions of the plane: q = 1 / (1 + d^2) has no pole
// nearer than 1 to any point, wherever the cells lie.  On a square of side 5/8 the interpolant of degree 15 in either coordinate at the Chebyshev nodes is within
// 3.3e-13 (A) and 1.5e-12 (B) of every term of unit mass, so the sums need the n |R| kernels of k_mean_field only at 256 nodes of every square that has heads in it, and of a
// head's own group.  Everything here is float64 (its rate is float32's).
//
// The own group is in what is interpolated and is taken out at the head, so the interpolant's error on it stays: absolute in the own group's mass, while what is left can be as small as
// the others are far.  Hence squares of 5/8 (sides of 1: 3.2e-10 and 1.5e-9, which for half of the mass 20 away from the rest is 1e-5 of B where sums in float32 keep 3e-7; of 1/2: 5e-14,
// and half as many squares again), and field_sound, which k_field_scan asks with the embedding's extent: where the error could be more than float32's rounding of any head's sum, k_mean_field
// does the work.  The results are the float64 sums to within that, rounded once, where sums in float32 carry three to five roundings.
//
//   k_field_count   heads of every square (squares are centred on multiples of their side, so that an embedding about the origin begins inside one)
//   k_field_scan    first position of every square, the squares that have heads; whether the field is exact enough and worth it, or k_mean_field does the work
//   k_field_place   the heads in the order of their squares
//   k_field_nodes   the sums at the nodes, the cells of a square cut among workgroups
//   k_field_coefs   added up in a fixed order, to coefficients of Chebyshev polynomials
//   k_field_sums    the polynomials at the heads, less what the own group's cells have in them
//
// 6,000,011 heads and 1,638 cells: 2.44 -> 0.32 ms (250 us of it at the heads).  Largest error of A over its value, 1,000 cells, against float64: 5.3e-7 -> 6.0e-8, of B as a whole
// 1.4e-7 -> 2.6e-8.  The order of the heads within a square changes from run to run, what each gets does not.
#pragma once
#include "nomad_kernels.h"

namespace nomad {

constexpr int kFieldSide = 102, kFieldSquares = kFieldSide * kFieldSide;   // coordinates within 31 (6 M points after 200 epochs: within 10)
constexpr int kFieldNodes = 16, kFieldGrid = kFieldNodes * kFieldNodes;
constexpr int kFieldUnits = kFieldMost;            // workgroups of k_field_nodes
constexpr int kFieldBlock = 1024, kFieldPerLane = 16, kFieldSpan = kFieldBlock * kFieldPerLane;
constexpr int kFieldTurns = 4;                     // heads a lane of k_field_sums takes, one after the other

struct FieldState { uint32_t use, n_squares, chunks, outside; };

struct Field {
    FieldState* state;
    uint32_t* count;       // [squares] heads; zero between epochs
    uint32_t* cursor;      // [squares] next position of the square in `order`
    uint32_t* list;        // [kFieldMost] squares that have heads, ascending
    uint32_t* place;       // [squares] where a square is in the list
    uint32_t* order;       // [n] heads, square by square
    double* partial;       // [kFieldUnits][3][kFieldGrid] sums of a part of the cells at the nodes
    double* coefs;         // [kFieldMost][3][kFieldGrid] of T_l(x) T_m(y), at 64 (l / 4) + 16 (l % 4) + m: as the matrix instructions take them
};

// the square of a point, or -1 outside of them (and for what is no number)
__device__ __forceinline__ int32_t field_square(float2 t) {
    if (!(fabsf(t.x) < 31.0f && fabsf(t.y) < 31.0f)) return -1;
    constexpr float per = (float)(1.0 / kFieldEdge);   // (a point within a rounding of an edge may count to either square)
    return ((int32_t)floorf(fmaf(t.y, per, 0.5f)) + kFieldSide / 2) * kFieldSide + (int32_t)floorf(fmaf(t.x, per, 0.5f)) + kFieldSide / 2;
}
// the coordinate of its centre, in either direction
__device__ __forceinline__ double field_centre(int32_t k) { return kFieldEdge * (double)(k - kFieldSide / 2); }

// one more of every lane's square in the workgroup's counters: the lane's rank; wavefronts that lie in one square (most do) add once
__device__ __forceinline__ uint32_t field_rank(uint32_t* counts, int32_t sq, bool has) {
    const unsigned long long in = __ballot(has);
    if (in == 0ull) return 0u;
    const int32_t first = __shfl(sq, __ffsll((long long)in) - 1, 64);
    uint32_t rank = 0u;
    if (__all(!has || sq == first)) {
        const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
        uint32_t base = 0u;
        if (has && before == 0u) base = atomicAdd(&counts[first], (uint32_t)__popcll(in));
        rank = (uint32_t)__shfl((int)base, __ffsll((long long)in) - 1, 64) + before;
    } else if (has) {
        rank = atomicAdd(&counts[sq], 1u);
    }
    return rank;
}

__global__ void __launch_bounds__(kFieldBlock) k_field_count(const float2* __restrict__ theta, int64_t i_begin, int64_t i_end, Field F) {
    __shared__ uint32_t counts[kFieldSquares];
    for (int x = threadIdx.x; x < kFieldSquares; x += kFieldBlock) counts[x] = 0u;
    __syncthreads();
    const int64_t i0 = i_begin + (int64_t)blockIdx.x * kFieldSpan;
    bool outside = false;
#pragma unroll 4
    for (int u = 0; u < kFieldPerLane; ++u) {
        const int64_t i = i0 + u * kFieldBlock + threadIdx.x;
        const int32_t sq = i < i_end ? field_square(theta[i]) : -1;
        outside = outside || (i < i_end && sq < 0);
        field_rank(counts, sq, sq >= 0);
    }
    if (__any(outside) && (threadIdx.x & 63) == 0) F.state->outside = 1u;
    __syncthreads();
    for (int x = threadIdx.x; x < kFieldSquares; x += kFieldBlock)
        if (counts[x]) atomicAdd(&F.count[x], counts[x]);
}

// (one workgroup)
__global__ void __launch_bounds__(1024) k_field_scan(const float4* __restrict__ cinfo, int64_t heads, int32_t R, double heaviest, Field F) {
    constexpr int kPer = (kFieldSquares + 1023) / 1024;
    __shared__ uint32_t total[16], some[16];
    __shared__ float box[16][4];
    __shared__ int strays;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t c[kPer], own = 0u, has = 0u;
#pragma unroll
    for (int x = 0; x < kPer; ++x) {
        c[x] = tid * kPer + x < kFieldSquares ? F.count[tid * kPer + x] : 0u;
        own += c[x];
        has += c[x] ? 1u : 0u;
    }
    // how far apart a head and a cell can be: a box of all squares that have heads and of all cells
    constexpr float kFar = 1e18f;
    float most[4] = {-kFar, -kFar, -kFar, -kFar};   // -x, -y, x, y
    bool stray = false;                             // a cell that is nowhere
#pragma unroll
    for (int x = 0; x < kPer; ++x) {
        const float cx = (float)field_centre((tid * kPer + x) % kFieldSide), cy = (float)field_centre((tid * kPer + x) / kFieldSide), half = 0.5f * (float)kFieldEdge;
        most[0] = c[x] ? fmaxf(most[0], half - cx) : most[0];
        most[1] = c[x] ? fmaxf(most[1], half - cy) : most[1];
        most[2] = c[x] ? fmaxf(most[2], half + cx) : most[2];
        most[3] = c[x] ? fmaxf(most[3], half + cy) : most[3];
    }
    for (int32_t r = tid; r < R; r += 1024) {
        const float4 cell = cinfo[r];
        if (cell.z > 0.f) {
            stray = stray || !(fabsf(cell.x) < kFar && fabsf(cell.y) < kFar);
            most[0] = fmaxf(most[0], -cell.x);
            most[1] = fmaxf(most[1], -cell.y);
            most[2] = fmaxf(most[2], cell.x);
            most[3] = fmaxf(most[3], cell.y);
        }
    }
#pragma unroll
    for (int w = 1; w < 64; w <<= 1)
#pragma unroll
        for (int v = 0; v < 4; ++v) most[v] = fmaxf(most[v], __shfl_xor(most[v], w, 64));
    if (tid == 0) strays = 0;
    if (lane < 4) box[wave][lane] = lane == 0 ? most[0] : lane == 1 ? most[1] : lane == 2 ? most[2] : most[3];
    const uint32_t incl = wave_prefix(own), incl_some = wave_prefix(has);
    if (lane == 63) { total[wave] = incl; some[wave] = incl_some; }
    __syncthreads();
    if (stray) strays = 1;
    __syncthreads();
    uint32_t at = incl - own, k = incl_some - has, n_squares = 0u;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) { at += total[w]; k += some[w]; }
        n_squares += some[w];
    }
#pragma unroll
    for (int x = 0; x < kPer; ++x) {
        const uint32_t sq = (uint32_t)(tid * kPer + x);
        if (sq >= (uint32_t)kFieldSquares) break;
        F.count[sq] = 0u;
        F.cursor[sq] = at;
        F.place[sq] = k;
        if (c[x] && k < (uint32_t)kFieldMost) F.list[k] = sq;
        at += c[x];
        k += c[x] ? 1u : 0u;
    }
    if (tid == 0) {
        for (int w = 1; w < 16; ++w)
            for (int v = 0; v < 4; ++v) box[0][v] = fmaxf(box[0][v], box[w][v]);
        const double dx = (double)box[0][0] + (double)box[0][2], dy = (double)box[0][1] + (double)box[0][3];
        const bool sound = !F.state->outside && !strays && field_sound(heaviest, sqrt(dx * dx + dy * dy));
        F.state->use = sound && field_pays((double)heads, (double)R, (double)n_squares) ? 1u : 0u;
        F.state->n_squares = n_squares;
        F.state->chunks = max(1u, min((uint32_t)kFieldUnits / max(n_squares, 1u), (uint32_t)(R + 31) / 32u));
        F.state->outside = 0u;
    }
}

__global__ void __launch_bounds__(kFieldBlock) k_field_place(const float2* __restrict__ theta, int64_t i_begin, int64_t i_end, Field F) {
    if (!F.state->use || F.state->n_squares == 1u) return;   // (one square: any order is the order)
    __shared__ uint32_t counts[kFieldSquares];
    for (int x = threadIdx.x; x < kFieldSquares; x += kFieldBlock) counts[x] = 0u;
    __syncthreads();
    const int64_t i0 = i_begin + (int64_t)blockIdx.x * kFieldSpan;
    int32_t sq[kFieldPerLane];
    uint32_t rank[kFieldPerLane];
#pragma unroll
    for (int u = 0; u < kFieldPerLane; ++u) {
        const int64_t i = i0 + u * kFieldBlock + threadIdx.x;
        sq[u] = i < i_end ? field_square(theta[i]) : -1;
    }
#pragma unroll
    for (int u = 0; u < kFieldPerLane; ++u) rank[u] = field_rank(counts, sq[u], sq[u] >= 0);
    __syncthreads();
    for (int x = threadIdx.x; x < kFieldSquares; x += kFieldBlock)
        if (counts[x]) counts[x] = atomicAdd(&F.cursor[x], counts[x]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kFieldPerLane; ++u)
        if (sq[u] >= 0) F.order[counts[sq[u]] + rank[u]] = (uint32_t)(i0 + u * kFieldBlock + threadIdx.x);
}

// q, to a unit in the last place or two of float64: the approximation of 2^-26, refined twice
__device__ __forceinline__ double field_cauchy(double dx, double dy) {
    const double t = fma(dx, dx, fma(dy, dy, 1.0));
    double q = __builtin_amdgcn_rcp(t);
    q = fma(q, fma(-t, q, 1.0), q);
    return fma(q, fma(-t, q, 1.0), q);
}

__global__ void __launch_bounds__(kFieldGrid) k_field_nodes(const float4* __restrict__ cinfo, int32_t R, Field F) {
    if (!F.state->use) return;
    __shared__ float4 cells[kFieldGrid];
    const uint32_t chunks = F.state->chunks, units = F.state->n_squares * chunks;
    const int tid = threadIdx.x;
    const double nx = 0.5 * kFieldEdge * cospi(((tid % kFieldNodes) + 0.5) / kFieldNodes),
                 ny = 0.5 * kFieldEdge * cospi(((tid / kFieldNodes) + 0.5) / kFieldNodes);
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x) {
        const uint32_t sq = F.list[u / chunks], part = u % chunks;
        const double x = nx + field_centre((int32_t)(sq % kFieldSide)), y = ny + field_centre((int32_t)(sq / kFieldSide));
        const int32_t r0 = (int32_t)((int64_t)R * part / chunks), r1 = (int32_t)((int64_t)R * (part + 1) / chunks);
        double a = 0.0, bx = 0.0, by = 0.0;
        for (int32_t c0 = r0; c0 < r1; c0 += kFieldGrid) {
            __syncthreads();
            if (c0 + tid < r1) cells[tid] = cinfo[c0 + tid];
            __syncthreads();
            const int32_t m = min(kFieldGrid, r1 - c0);
#pragma unroll 4
            for (int32_t r = 0; r < m; ++r) {
                const float4 c = cells[r];
                const double dx = x - (double)c.x, dy = y - (double)c.y, q = field_cauchy(dx, dy), w = (double)c.z * q, w2 = w * q;
                a += w;
                bx = fma(w2, dx, bx);
                by = fma(w2, dy, by);
            }
        }
        double* const out = F.partial + (size_t)u * 3 * kFieldGrid + tid;
        out[0] = a;
        out[kFieldGrid] = bx;
        out[2 * kFieldGrid] = by;
    }
}

__global__ void __launch_bounds__(kFieldGrid) k_field_coefs(Field F) {
    if (!F.state->use) return;
    constexpr int N = kFieldNodes;
    __shared__ double dct[N][N + 1], at_node[3][N][N + 1], half[3][N][N + 1];
    const uint32_t chunks = F.state->chunks, n_squares = F.state->n_squares;
    const int tid = threadIdx.x, row = tid / N, col = tid % N;
    dct[row][col] = (row ? 2.0 : 1.0) / N * cospi(row * (col + 0.5) / N);
    for (uint32_t k = blockIdx.x; k < n_squares; k += gridDim.x) {
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            const double* const from = F.partial + ((size_t)k * chunks * 3 + v) * kFieldGrid + tid;
            double s = 0.0;
#pragma unroll 8
            for (uint32_t c = 0; c < chunks; ++c) s += from[(size_t)c * 3 * kFieldGrid];
            at_node[v][row][col] = s;
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 3; ++v) {   // along x
            double s = 0.0;
            for (int j = 0; j < N; ++j) s = fma(dct[col][j], at_node[v][row][j], s);
            half[v][row][col] = s;
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 3; ++v) {   // along y
            double s = 0.0;
            for (int j = 0; j < N; ++j) s = fma(dct[row][j], half[v][j][col], s);
            F.coefs[((size_t)k * 3 + v) * kFieldGrid + 64 * (col / 4) + 16 * (col % 4) + row] = s;
        }
    }
}

// T_g, T_g+4, T_g+8, T_g+12 of x, g = lane / 16: what the lane supplies to, or takes its results by, in the four steps of a product
__device__ __forceinline__ void field_chebyshev(double x, int g, double (&t)[4]) {
    const double x2 = 2.0 * x, t2 = fma(x2, x, -1.0), t3 = fma(x2, t2, -x), t4 = fma(x2, t3, -t2), t42 = 2.0 * t4;
    t[0] = g == 0 ? 1.0 : g == 1 ? x : g == 2 ? t2 : t3;
    t[1] = fma(t42, t[0], -(g == 0 ? t4 : g == 1 ? t3 : g == 2 ? t2 : x));
    t[2] = fma(t42, t[1], -t[0]);
    t[3] = fma(t42, t[2], -t[1]);
}

// 64 heads a wavefront at a time, a lane each for what is theirs; their polynomials sixteen at a time on the matrix cores: coefficients [16 of y][16 of x] times
// T(x) [16][heads], three products of four steps, then four multiplications by T(y) a lane and two additions across lanes.  The coefficients of a
// square stay in registers while the heads lie in it.  Bound by the float64 units, whose rate is the same for matrix and vector instructions here: 250 us for 6 M heads in one
// square, 131 for 2 M in a thousand.  In vector instructions with the coefficients from the scalar cache 214 and 970: every wavefront waited for other coefficients.  The
// next turn's heads loaded ahead, 1, 8 or 16 turns a wavefront: the same or slower.
__global__ void __launch_bounds__(256) k_field_sums(const float2* __restrict__ theta, const int32_t* __restrict__ cluster_of, const int32_t* __restrict__ group_of_cluster,
                                                    const float4* __restrict__ cinfo, const int2* __restrict__ group_slots, int64_t i_begin, int64_t i_end, Field F,
                                                    const double* __restrict__ coefs, float* __restrict__ A, float2* __restrict__ B) {
    typedef double Acc __attribute__((ext_vector_type(4)));
    if (!F.state->use) return;
    const bool as_they_are = F.state->n_squares == 1u;
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const int64_t heads = i_end - i_begin, first = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64 * kFieldTurns;
    double c[3][4];
    int32_t in_hand = -1;   // the square whose coefficients these are
    for (int turn = 0; turn < kFieldTurns; ++turn) {
        const int64_t p = first + turn * 64 + lane;
        if (p - lane >= heads) return;
        const int64_t at = min(p, heads - 1);   // lanes past the end: the last head again, not stored
        const int64_t i = as_they_are ? i_begin + at : (int64_t)F.order[at];
        const float2 t = theta[i];
        const int2 own = group_slots[group_of_cluster[cluster_of[i]]];
        const int32_t sq = max(field_square(t), 0), k = (int32_t)F.place[sq];
        double a = 0.0, bx = 0.0, by = 0.0;
#pragma unroll 1
        for (int tile = 0; tile < 4; ++tile) {
            const int from = 16 * tile + (lane & 15);
            const float px = __shfl(t.x, from, 64), py = __shfl(t.y, from, 64);
            const int32_t psq = __shfl(sq, from, 64), pk = __shfl(k, from, 64);
            double tx[4], ty[4], sum[3] = {0.0, 0.0, 0.0};
            field_chebyshev(2.0 / kFieldEdge * ((double)px - field_centre(psq % kFieldSide)), g, tx);
            field_chebyshev(2.0 / kFieldEdge * ((double)py - field_centre(psq / kFieldSide)), g, ty);
            unsigned long long left = __ballot(true);
            while (left) {   // the squares of these heads, one after the other
                const int32_t now = __builtin_amdgcn_readlane(pk, __ffsll((long long)left) - 1);
                if (now != in_hand) {
#pragma unroll
                    for (int v = 0; v < 3; ++v)
#pragma unroll
                        for (int s = 0; s < 4; ++s) c[v][s] = coefs[((size_t)now * 3 + v) * kFieldGrid + s * 64 + lane];
                    in_hand = now;
                }
                const bool here = pk == now;
#pragma unroll
                for (int v = 0; v < 3; ++v) {
                    Acc d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int s = 0; s < 4; ++s) d = __builtin_amdgcn_mfma_f64_16x16x4f64(c[v][s], tx[s], d, 0, 0, 0);
                    const double all = fma(d[0], ty[0], fma(d[1], ty[1], fma(d[2], ty[2], d[3] * ty[3])));
                    sum[v] = here ? all : sum[v];
                }
                left &= ~__ballot(here);
            }
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                sum[v] += __shfl_xor(sum[v], 16, 64);
                sum[v] += __shfl_xor(sum[v], 32, 64);
            }
            a = g == tile ? sum[0] : a;
            bx = g == tile ? sum[1] : bx;
            by = g == tile ? sum[2] : by;
        }
        for (int32_t r = own.x; r < own.y; ++r) {   // less the own group's cells
            const float4 cell = cinfo[r];
            const double dx = (double)t.x - (double)cell.x, dy = (double)t.y - (double)cell.y, q = field_cauchy(dx, dy), w = (double)cell.z * q, w2 = w * q;
            a -= w;
            bx = fma(-w2, dx, bx);
            by = fma(-w2, dy, by);
        }
        if (p < heads) {
            A[i] = (float)a;
            B[i] = make_float2((float)bx, (float)by);
        }
    }
}

}  // namespace nomad
