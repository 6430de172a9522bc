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
//   k_field_lay     the sums at the nodes, a square's cells cut among workgroups; the heads in the order of their squares
//   k_field_coefs   added up, to coefficients of Chebyshev polynomials
//   k_field_sums    the polynomials at the heads, less what the own group's cells have in them
//
// An embedding that the field cannot use pays for the launches all the same: 500,000 heads and 1,050 cells 145 -> 173 us (178 with a launch for nodes and places each and longer spans of heads).
//
// 6,000,011 heads and 1,638 cells: 2.36 -> 0.28 ms in one square (220 us of it at the heads), 0.59 in 1,290.  Largest error of A over its value, 1,000 cells, against float64: 5.3e-7 -> 6.0e-8, of B as a whole
// 1.4e-7 -> 2.6e-8.  The order of the heads within a square changes from run to run, what each gets does not.
#pragma once
#include "nomad_kernels.h"

namespace nomad {

constexpr int kFieldSide = 102, kFieldSquares = kFieldSide * kFieldSide;   // coordinates within 31 (6 M points after 200 epochs: within 10)
constexpr int kFieldTable = 12 * 1024;             // entries of a table of squares: twelve a lane of k_field_scan
static_assert(kFieldSquares <= kFieldTable, "");
constexpr int kFieldNodes = 16, kFieldGrid = kFieldNodes * kFieldNodes;
constexpr int kFieldParts = 2048;                  // workgroups' worth of nodes: parts of the cells of every square, where the squares are fewer (eight for every unit: they are not all as long)
constexpr int kFieldUnits = kFieldMost > kFieldParts ? kFieldMost : kFieldParts;   // (square, part of the cells) pairs
constexpr int kFieldPartCells = 256;               // cells a part has at least, where it is not all
constexpr int kFieldCountBlock = 1024, kFieldLayBlock = 512, kFieldLayWaves = kFieldLayBlock / 64, kFieldNodeBlocks = 512;
constexpr int kFieldFewHeads = 2 << 20, kFieldFew = 4, kFieldMany = 16;   // heads a lane of the counting pass has, below and above: workgroups for all units below
inline int64_t field_count_span(int64_t heads) { return kFieldCountBlock * (heads < kFieldFewHeads ? kFieldFew : kFieldMany); }
inline int64_t field_place_span(int64_t heads) { return kFieldLayBlock * (heads < kFieldFewHeads ? kFieldFew : kFieldMany); }
constexpr int kFieldTurns = 4;                     // heads a lane of k_field_sums takes, one after the other

struct FieldState { uint32_t use, n_squares, chunks, outside; };   // outside: zero between epochs

struct Field {
    FieldState* state;
    uint32_t* count;       // [kFieldTable] heads of a square; zero between epochs
    uint32_t* cursor;      // [kFieldTable] next position of the square in `order`
    uint32_t* list;        // [kFieldMost] squares that have heads, ascending
    uint32_t* place;       // [kFieldTable] where a square is in the list
    uint32_t* order;       // [n] heads, square by square
    double* partial;       // [kFieldUnits][3][kFieldGrid] sums of a part of the cells at the nodes, (x, y) at 64 (x / 4) + 16 (x % 4) + y
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

template <int PER>
__global__ void __launch_bounds__(kFieldCountBlock, 8) k_field_count(const float2* __restrict__ theta, int64_t i_begin, int64_t i_end, Field F) {
    __shared__ uint32_t counts[kFieldSquares];
    for (int x = threadIdx.x; x < kFieldSquares; x += kFieldCountBlock) counts[x] = 0u;
    __syncthreads();
    const int64_t i0 = i_begin + (int64_t)blockIdx.x * (kFieldCountBlock * PER);
    bool outside = false;
#pragma unroll 4
    for (int u = 0; u < PER; ++u) {
        const int64_t i = i0 + u * kFieldCountBlock + threadIdx.x;
        const int32_t sq = i < i_end ? field_square(theta[i]) : -1;
        outside = outside || (i < i_end && sq < 0);
        field_rank(counts, sq, sq >= 0);
    }
    if (__any(outside) && (threadIdx.x & 63) == 0) F.state->outside = 1u;
    __syncthreads();
    for (int x = threadIdx.x; x < kFieldSquares; x += kFieldCountBlock)
        if (counts[x]) atomicAdd(&F.count[x], counts[x]);
}

// (one workgroup)
__global__ void __launch_bounds__(1024) k_field_scan(const float4* __restrict__ cinfo, int64_t heads, int32_t R, double heaviest, Field F) {
    constexpr int kPer = kFieldTable / 1024;
    __shared__ uint32_t total[16], some[16];
    __shared__ float box[16][4];
    __shared__ int strays;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t c[kPer], own = 0u, has = 0u;
    uint4* const mine = (uint4*)F.count + tid * (kPer / 4);
#pragma unroll
    for (int x = 0; x < kPer; x += 4) {
        const uint4 four = mine[x / 4];
        mine[x / 4] = make_uint4(0u, 0u, 0u, 0u);
        c[x] = four.x; c[x + 1] = four.y; c[x + 2] = four.z; c[x + 3] = four.w;
    }
#pragma unroll
    for (int x = 0; x < kPer; ++x) {
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
    uint32_t first[kPer], place[kPer];
#pragma unroll
    for (int x = 0; x < kPer; ++x) {
        first[x] = at;
        place[x] = k;
        if (c[x] && k < (uint32_t)kFieldMost) F.list[k] = (uint32_t)(tid * kPer + x);
        at += c[x];
        k += c[x] ? 1u : 0u;
    }
#pragma unroll
    for (int x = 0; x < kPer; x += 4) {
        ((uint4*)F.cursor)[tid * (kPer / 4) + x / 4] = make_uint4(first[x], first[x + 1], first[x + 2], first[x + 3]);
        ((uint4*)F.place)[tid * (kPer / 4) + x / 4] = make_uint4(place[x], place[x + 1], place[x + 2], place[x + 3]);
    }
    if (tid == 0) {
        for (int w = 1; w < 16; ++w)
            for (int v = 0; v < 4; ++v) box[0][v] = fmaxf(box[0][v], box[w][v]);
        const double dx = (double)box[0][0] + (double)box[0][2], dy = (double)box[0][1] + (double)box[0][3];
        const bool sound = !F.state->outside && !strays && field_sound(heaviest, sqrt(dx * dx + dy * dy));
        F.state->use = sound && field_pays((double)heads, (double)R, (double)n_squares) ? 1u : 0u;
        F.state->n_squares = n_squares;
        F.state->chunks = max(1u, min((uint32_t)kFieldParts / max(n_squares, 1u), (uint32_t)(R + kFieldPartCells - 1) / kFieldPartCells));
        F.state->outside = 0u;
    }
}

// 1 / t, to a unit in the last place or two of float64: the approximation of 2^-23 and better, refined once by a cubic step
__device__ __forceinline__ double field_reciprocal(double t) {
    const double q = __builtin_amdgcn_rcp(t), e = fma(-t, q, 1.0);
    return fma(q, fma(e, e, e), q);
}

// The sums at the nodes: a workgroup takes a part of the cells for one square, a wavefront an eighth of those for all 256 nodes, four a lane ((x, y) with x = lane / 16
// + 0, 4, 8, 12 and y = lane % 16), whose differences in y and whose reciprocal it shares: 13 float64 instructions a cell and node where a lane for each node had 20, and no barrier among the
// cells.  Eight wavefronts' sums are added in LDS, in a fixed order.  250,003 heads in 221 squares, 2,100 cells: 61 us with the places, 1.9 times
// what the instructions take (a lane for each node, with barriers: 85, and 18 for the places); 6 M heads in 1,290 squares, 1,638 cells 256.
__device__ __forceinline__ void field_nodes(const float4* __restrict__ cinfo, int32_t R, const Field& F, double (&sums)[kFieldLayWaves / 2][12][64]) {
    constexpr int N = kFieldNodes;
    const uint32_t chunks = F.state->chunks, units = F.state->n_squares * chunks;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15, g = lane >> 4;
    double nx[4];
    const double ny = 0.5 * kFieldEdge * cospi((col + 0.5) / N);
#pragma unroll
    for (int s = 0; s < 4; ++s) nx[s] = 0.5 * kFieldEdge * cospi((4 * s + g + 0.5) / N);
    for (uint32_t u = blockIdx.x; u < units; u += kFieldNodeBlocks) {
        const uint32_t k = u / chunks, part = u % chunks, sq = F.list[k];
        const double y = ny + field_centre((int32_t)(sq / kFieldSide)), x0 = field_centre((int32_t)(sq % kFieldSide));
        const int64_t cuts = (int64_t)chunks * kFieldLayWaves, cut = (int64_t)part * kFieldLayWaves + wave;
        const int32_t r0 = (int32_t)(R * cut / cuts), r1 = (int32_t)(R * (cut + 1) / cuts);
        double v[3][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) v[0][s] = v[1][s] = v[2][s] = 0.0;
#pragma unroll 2
        for (int32_t r = r0; r < r1; ++r) {
            const float4 c = cinfo[r];
            const double dy = y - (double)c.y, y2 = fma(dy, dy, 1.0), from = x0 - (double)c.x, p = (double)c.z;
            double dx[4], t[4], q[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) { dx[s] = nx[s] + from; t[s] = fma(dx[s], dx[s], y2); }
            const double t01 = t[0] * t[1], t23 = t[2] * t[3], i = field_reciprocal(t01 * t23), i01 = i * t23, i23 = i * t01;
            q[0] = i01 * t[1]; q[1] = i01 * t[0]; q[2] = i23 * t[3]; q[3] = i23 * t[2];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double w = p * q[s], w2 = w * q[s];
                v[0][s] += w;
                v[1][s] = fma(w2, dx[s], v[1][s]);
                v[2][s] = fma(w2, dy, v[2][s]);
            }
        }
#pragma unroll
        for (int half = kFieldLayWaves / 2; half > 0; half >>= 1) {
            if (wave >= half && wave < 2 * half)
#pragma unroll
                for (int m = 0; m < 12; ++m) sums[wave - half][m][lane] = v[m / 4][m % 4];
            __syncthreads();
            if (wave < half)
#pragma unroll
                for (int m = 0; m < 12; ++m) v[m / 4][m % 4] += sums[wave][m][lane];
            __syncthreads();
        }
        if (wave > 0) continue;
        double* const out = F.partial + (size_t)u * 3 * kFieldGrid + lane;
#pragma unroll
        for (int m = 0; m < 12; ++m) out[64 * m] = v[m / 4][m % 4];
    }
}

template <int PER>
__device__ __forceinline__ void field_place(const float2* __restrict__ theta, int64_t i_begin, int64_t i_end, uint32_t block, const Field& F, uint32_t (&counts)[kFieldSquares]) {
    for (int x = threadIdx.x; x < kFieldSquares; x += kFieldLayBlock) counts[x] = 0u;
    __syncthreads();
    const int64_t i0 = i_begin + (int64_t)block * (kFieldLayBlock * PER);
    int32_t sq[PER];
    uint32_t rank[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t i = i0 + u * kFieldLayBlock + threadIdx.x;
        sq[u] = i < i_end ? field_square(theta[i]) : -1;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) rank[u] = field_rank(counts, sq[u], sq[u] >= 0);
    __syncthreads();
    for (int x = threadIdx.x; x < kFieldSquares; x += kFieldLayBlock)
        if (counts[x]) counts[x] = atomicAdd(&F.cursor[x], counts[x]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (sq[u] >= 0) F.order[counts[sq[u]] + rank[u]] = (uint32_t)(i0 + u * kFieldLayBlock + threadIdx.x);
}

// workgroups: kFieldNodeBlocks for the nodes, then one a span of heads to be placed
template <int PER>
__global__ void __launch_bounds__(kFieldLayBlock) k_field_lay(const float2* __restrict__ theta, const float4* __restrict__ cinfo, int64_t i_begin, int64_t i_end, int32_t R,
                                                              Field F) {
    if (!F.state->use) return;
    __shared__ union { double sums[kFieldLayWaves / 2][12][64]; uint32_t counts[kFieldSquares]; } lds;
    if (blockIdx.x < (uint32_t)kFieldNodeBlocks) field_nodes(cinfo, R, F, lds.sums);
    else if (F.state->n_squares > 1u) field_place<PER>(theta, i_begin, i_end, blockIdx.x - (uint32_t)kFieldNodeBlocks, F, lds.counts);   // (one square: any order is the order)
}

// The parts of a square added up in a fixed order and turned to coefficients on the matrix cores, a square a wavefront: the operands lie as the lanes hold the sums, and the product
// along x is the operand of the one along y.
__global__ void __launch_bounds__(256) k_field_coefs(Field F) {
    typedef double Acc __attribute__((ext_vector_type(4)));
    const uint32_t chunks = F.state->chunks, k = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (!F.state->use || k >= F.state->n_squares) return;
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    double dct[4], v[3][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        dct[s] = (col ? 2.0 : 1.0) / kFieldNodes * cospi(col * (4 * s + g + 0.5) / kFieldNodes);
        v[0][s] = v[1][s] = v[2][s] = 0.0;
    }
    const double* const from = F.partial + (size_t)k * chunks * 3 * kFieldGrid + lane;
#pragma unroll 2
    for (uint32_t c = 0; c < chunks; ++c)
#pragma unroll
        for (int m = 0; m < 12; ++m) v[m / 4][m % 4] += from[(size_t)c * 3 * kFieldGrid + 64 * m];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        Acc h = {0.0, 0.0, 0.0, 0.0}, d = h;
#pragma unroll
        for (int s = 0; s < 4; ++s) h = __builtin_amdgcn_mfma_f64_16x16x4f64(v[m][s], dct[s], h, 0, 0, 0);   // [y][T of x]
#pragma unroll
        for (int s = 0; s < 4; ++s) d = __builtin_amdgcn_mfma_f64_16x16x4f64(h[s], dct[s], d, 0, 0, 0);      // [T of x][T of y]
#pragma unroll
        for (int s = 0; s < 4; ++s) F.coefs[((size_t)k * 3 + m) * kFieldGrid + 64 * s + lane] = d[s];
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
            const double dx = (double)t.x - (double)cell.x, dy = (double)t.y - (double)cell.y, q = field_reciprocal(fma(dx, dx, fma(dy, dy, 1.0))), w = (double)cell.z * q,
                         w2 = w * q;
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
