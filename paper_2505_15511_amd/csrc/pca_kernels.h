// Device code of the PCA initialisation (Section 3.5: the projection starts from a PCA of the data).
//
//   shift       a = the mean of up to kShiftRows rows spread over the set, in float64: near the mean, so that
//   covariance  C = (1/n) sum_i (x_i - a)(x_i - a)^T - (mean - a)(mean - a)^T loses nothing: |mean - a|^2 is of the order of the
//               variance over the sampled rows, n / kShiftRows times the variance at the very worst (four digits of the sixteen).  A dense
//               contraction over the points, on the float64 matrix cores (v_mfma_f64_16x16x4f64), one wavefront per 64x64 tile
//               of C and slab of rows, slabs added in order; the tiles on the diagonal also add up the columns, for
//   mean        = a + (1/n) sum_i (x_i - a)
//   axes        the leading eigenvectors of C by subspace iteration accelerated with Chebyshev polynomials: a block of
//               kRitz vectors, a Rayleigh-Ritz step (the 8 x 8 pencil on one wavefront) after every polynomial
//   scores      theta_i = ((x_i - mean) . axis_1, (x_i - mean) . axis_2), float64, oriented and scaled, rounded once
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nomad_pca {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kShiftRows = 256;   // rows of the shift
constexpr int kColBlock = 64;     // a wavefront's tile of C is kColBlock x kColBlock (4 x 4 matrix-core tiles)
constexpr int kRitz = 8;          // vectors iterated together (convergence goes with lambda_9 / lambda_2)
constexpr int kMaxDim = 768;

// shift = mean of the m rows floor(i n / m); a workgroup per 64 columns, every wavefront its share of the rows (eight in flight)
constexpr int kMeanWaves = 16;
__global__ void __launch_bounds__(64 * kMeanWaves) k_pca_shift(const float* __restrict__ X, int64_t n, int32_t d, double* __restrict__ shift) {
    __shared__ double sum[kMeanWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = blockIdx.x * 64 + lane, c = min(col, d - 1);
    const int m = (int)min((int64_t)kShiftRows, n);
    double s = 0.0;
    for (int i = wave; i < m; i += 8 * kMeanWaves) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = X[(int64_t)min(i + u * kMeanWaves, m - 1) * n / m * d + c];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += i + u * kMeanWaves < m ? (double)v[u] : 0.0;
    }
    sum[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && col < d) {
        double t = 0.0;
        for (int w = 0; w < kMeanWaves; ++w) t += sum[w][lane];
        shift[col] = t / (double)m;
    }
}

// delta = sum of the slabs' column sums of x - shift / n, mean = shift + delta; a workgroup per 64 columns, every wavefront its share of
// the partial sums (eight in flight), the wavefronts' sums added in order.  (One thread per column took 31 us for 977 slabs.)
__global__ void __launch_bounds__(64 * kMeanWaves) k_pca_mean(const double* __restrict__ partial, int32_t blocks, int32_t d, int64_t n, const double* __restrict__ shift,
                                                              double* __restrict__ delta, double* __restrict__ mean) {
    __shared__ double sum[kMeanWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = blockIdx.x * 64 + lane;
    double s = 0.0;
    if (col < d) {
        int b = wave;
        for (; b + 7 * kMeanWaves < blocks; b += 8 * kMeanWaves) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = partial[(int64_t)(b + u * kMeanWaves) * d + col];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; b < blocks; b += kMeanWaves) s += partial[(int64_t)b * d + col];
    }
    sum[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && col < d) {
        double t = 0.0;
        for (int w = 0; w < kMeanWaves; ++w) t += sum[w][lane];
        t /= (double)n;
        delta[col] = t;
        mean[col] = shift[col] + t;
    }
}

// column blocks (a, b), a <= b, of tile pair number `pair` when there are nb column blocks: the diagonal first
__host__ __device__ inline void cov_pair(int pair, int nb, int& a, int& b) {
    if (pair < nb) { a = b = pair; return; }
    pair -= nb;
    a = 0;
    while (pair >= nb - 1 - a) { pair -= nb - 1 - a; ++a; }
    b = a + 1 + pair;
}

// Slabs of rows of a tile pair.  A tile on the diagonal takes 10 of the 16 products (the others are their mirror images), kDiagonalShare of the time:
// its slabs are longer, so that all the wavefronts end together.
constexpr double kDiagonalShare = 0.7;   // (with the columns' sums; million x 128: 0.56 0.343 ms, 0.62 0.341, 0.68 0.325, 0.75 0.329)
struct CovSlabs { int32_t diag, off; int64_t diag_rows, off_rows; };

// One wavefront: tile pair blockIdx.x / slabs, rows slab * slab_rows ...  Operand layout of the 16x16x4 float64
// instruction: lane l supplies A[i = l % 16][k = l / 16] and B[k = l / 16][j = l % 16]; it receives D[i = l / 16 + 4 v][j = l % 16]
// in element v.  Here k runs over four consecutive rows of X, i and j over columns: D += Xc^T Xc.
//
// Bound by issue: a step of four rows is 16 matrix instructions of 64 cycles, and vector instructions do not overlap float64
// matrix instructions, so the step carries nothing but its loads (uniform base + 32-bit lane offset), conversions and
// subtractions.  Columns beyond d are read as the last column (their entries of C are never stored), only the last step of a
// slab masks rows.  n = 1e6, d = 128: 0.43 ms = 57 TFLOP/s executed (0.56 ms with every element masked), 0.325 without the mirrored
// products and with the columns' sums (a pass of 0.083 ms before); n = 1e5, d = 768: 1.12 ms, now 1.06.
template <bool DIAGONAL>
__device__ __forceinline__ void cov_tile(const float* __restrict__ X, int64_t n, int32_t d, const double* __restrict__ mean, int a, int b,
                                         int64_t r0, int64_t r1, double* __restrict__ out, double* __restrict__ sums) {
    const int lane = threadIdx.x, lr = lane >> 4, lc = lane & 15;
    uint32_t offa[4], offb[4];     // elements from the step's first row
    double ma[4], mb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int ca = min(a * kColBlock + 16 * u + lc, d - 1), cb = min(b * kColBlock + 16 * u + lc, d - 1);
        offa[u] = (uint32_t)(lr * d + ca);
        offb[u] = (uint32_t)(lr * d + cb);
        ma[u] = mean[ca];
        mb[u] = mean[cb];
    }
    doublex4 acc[4][4];
    double colsum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[x][y] = doublex4{0.0, 0.0, 0.0, 0.0};
    // loads run kAhead steps ahead of the multiplications: a step is about half a microsecond, and the rows come from HBM
    constexpr int kAhead = 4;
    const int64_t steps = (r1 - r0) / 4;
    float fa[kAhead][4], fb[kAhead][4];
    auto fetch = [&](int slot, int64_t step) {   // beyond the last step: the last step again (not used)
        const float* base = X + (r0 + 4 * min(step, steps - 1)) * d;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            fa[slot][u] = base[offa[u]];
            if (!DIAGONAL) fb[slot][u] = base[offb[u]];
        }
    };
    auto multiply = [&](const float (&va)[4], const float (&vb)[4], bool live) {
        double xa[4], xb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            xa[u] = live ? (double)va[u] - ma[u] : 0.0;
            xb[u] = DIAGONAL ? xa[u] : live ? (double)vb[u] - mb[u] : 0.0;
            if (DIAGONAL) colsum[u] += xa[u];
        }
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = DIAGONAL ? x : 0; y < 4; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[x], xb[y], acc[x][y], 0, 0, 0);
    };
    if (steps > 0) {
#pragma unroll
        for (int s = 0; s < kAhead; ++s) fetch(s, s);
        int64_t st = 0;
        for (; st + kAhead <= steps; st += kAhead) {
#pragma unroll
            for (int s = 0; s < kAhead; ++s) {   // slot s holds step st + s
                float va[4], vb[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) { va[u] = fa[s][u]; vb[u] = fb[s][u]; }
                fetch(s, st + s + kAhead);
                multiply(va, vb, true);
                __builtin_amdgcn_sched_barrier(0);   // left to itself the compiler converts four steps at once: one wavefront per SIMD
            }
        }
#pragma unroll
        for (int s = 0; s < kAhead; ++s)
            if (st + s < steps) multiply(fa[s], fb[s], true);
    }
    if (r0 + 4 * steps < r1) {   // one to three rows left
        const bool live = r0 + 4 * steps + lr < r1;
        const float* base = X + (r0 + 4 * steps) * d;
        float va[4], vb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            va[u] = live ? base[offa[u]] : 0.f;
            vb[u] = !DIAGONAL && live ? base[offb[u]] : 0.f;
        }
        multiply(va, vb, live);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = DIAGONAL ? x : 0; y < 4; ++y)
#pragma unroll
            for (int v = 0; v < 4; ++v) out[(16 * x + lr + 4 * v) * kColBlock + 16 * y + lc] = acc[x][y][v];
    if (DIAGONAL) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            double t = colsum[u];
            t += __shfl_xor(t, 16, 64);
            t += __shfl_xor(t, 32, 64);
            const int c = a * kColBlock + 16 * u + lc;
            if (lr == 0 && c < d) sums[c] = t;
        }
    }
}

// partial: [diagonal tiles][slabs.diag], then [the others][slabs.off] tiles; sums [slabs.diag][d]
__global__ void __launch_bounds__(64, 2) k_pca_cov(const float* __restrict__ X, int64_t n, int32_t d, const double* __restrict__ shift,
                                                CovSlabs slabs, double* __restrict__ partial, double* __restrict__ sums) {
    const int nb = (d + kColBlock - 1) / kColBlock, on_diag = nb * slabs.diag, rest = (int)blockIdx.x - on_diag;
    const int pair = rest < 0 ? (int)blockIdx.x / slabs.diag : nb + rest / slabs.off, slab = rest < 0 ? (int)blockIdx.x % slabs.diag : rest % slabs.off;
    int a, b;
    cov_pair(pair, nb, a, b);
    const int64_t rows = rest < 0 ? slabs.diag_rows : slabs.off_rows, r0 = min(n, (int64_t)slab * rows), r1 = min(n, r0 + rows);
    double* out = partial + (int64_t)blockIdx.x * (kColBlock * kColBlock);
    if (a == b) cov_tile<true>(X, n, d, shift, a, b, r0, r1, out, sums + (int64_t)slab * d);
    else cov_tile<false>(X, n, d, shift, a, b, r0, r1, out, nullptr);
}

// C = (1/n) sum over the slabs - delta delta^T; both triangles written.  A workgroup takes 32 consecutive entries of a tile, eight threads
// each: every eighth slab (eight in flight), the eight sums added in order.  (One thread per entry: 40 us for 683 slabs.)
constexpr int kReduceEntries = 32;
__global__ void __launch_bounds__(256) k_pca_cov_reduce(const double* __restrict__ partial, CovSlabs cut, int32_t d, int64_t n, const double* __restrict__ delta,
                                                        double* __restrict__ C) {
    __shared__ double part[8][kReduceEntries];
    const int sub = threadIdx.x / kReduceEntries, lane = threadIdx.x % kReduceEntries;
    const int64_t x = (int64_t)blockIdx.x * kReduceEntries + lane;   // kReduceEntries divides a tile: one pair per workgroup
    const int pair = (int)(x / (kColBlock * kColBlock)), e = (int)(x % (kColBlock * kColBlock));
    const int nb = (d + kColBlock - 1) / kColBlock, slabs = pair < nb ? cut.diag : cut.off;
    const int64_t first = pair < nb ? (int64_t)pair * cut.diag : (int64_t)nb * cut.diag + (int64_t)(pair - nb) * cut.off;
    const int row = e / kColBlock, column = e % kColBlock;
    const bool mirrored = pair < nb && row / 16 > column / 16;   // not computed: written with its mirror image
    double s = 0.0;
    const double* src = partial + first * (kColBlock * kColBlock) + e;
    int sl = mirrored ? slabs : sub;
    for (; sl + 56 < slabs; sl += 64) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(int64_t)(sl + 8 * u) * (kColBlock * kColBlock)];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; sl < slabs; sl += 8) s += src[(int64_t)sl * (kColBlock * kColBlock)];
    part[sub][lane] = s;
    __syncthreads();
    if (sub != 0 || mirrored) return;
    s = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) s += part[u][lane];
    int a, b;
    cov_pair(pair, nb, a, b);
    const int gi = a * kColBlock + row, gj = b * kColBlock + column;
    if (gi >= d || gj >= d) return;
    s = s / (double)n - delta[gi] * delta[gj];
    C[(int64_t)gi * d + gj] = s;
    if (a != b || row / 16 < column / 16) C[(int64_t)gj * d + gi] = s;
}

// ---- the leading eigenvectors of C: subspace iteration on a block of kRitz vectors, Chebyshev polynomials of C as the power
// Rayleigh-Ritz on the block (ritz_step) gives the Ritz vectors R and values lam; the next block is T_deg((C - c) / e) R,
// T the Chebyshev polynomial of the interval [0, b] (c = e = b / 2) whose upper end b is the smallest Ritz value of the
// block: components with eigenvalues in the interval stay bounded by 1, those above it grow like cosh(deg acosh(2 lam / b - 1)).
// Where C^4 per step needed 28 steps of 139 us for a million points in 128 dimensions (and 40 at flatter spectra), five to
// eight steps of degree up to kMaxDegree do, with their 8 x 8 algebra on a whole wavefront.
constexpr int kMaxDegree = 20;
constexpr int kRitzThreads = 1024; // of the step by itself: one row of the block per thread
constexpr int kSmallDim = 128;     // up to here the whole iteration is one workgroup (k_pca_axes_small) ...
constexpr int kSmallThreads = 512; // ... of one wavefront per 16-row tile of C

struct RitzState {                 // what a step decides, for the host and for the next step
    double lam[kRitz];
    double resid;                  // max over the first two pairs of |C w - lam w| / lam_1
    double c, e;                   // centre and half width of the interval
    double best;                   // smallest residual so far, for the stall rule
    int32_t degree;                // of the polynomial that makes the next block
    int32_t stall;
    int32_t steps;
};

__device__ __forceinline__ double shfl_f64(double v, int lane) { return __shfl(v, lane, 64); }

// 1 / sqrt(x) and 1 / x of a normal number: the instruction's estimate (2^-14 at least) and Newton's steps, each of which squares
// the error: three leave only roundings.  (A square root and a division take several times as long, one after the other; with them
// in the pencil's factor and rotations the five steps of a million x 128 took 246 us, now 203.)
template <int NEWTON>
__device__ __forceinline__ double newton_rsqrt(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int i = 0; i < NEWTON; ++i) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return y;
}
template <int NEWTON>
__device__ __forceinline__ double newton_rcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int i = 0; i < NEWTON; ++i) y = fma(y, fma(-x, y, 1.0), y);
    return y;
}

// Eigenpairs of the pencil H w = lam G w (both symmetric kRitz x kRitz, G positive semi-definite) on one wavefront, matrix
// entry (i, j) in lane 8 i + j.  G is scaled to a unit diagonal and factored, G = L L^T; S = L^-1 H L^-T is diagonalised by
// Jacobi rotations, four disjoint ones at a time (seven rounds per sweep pair every index with every other).  A column
// whose pivot vanishes (dependent on the ones before it, or absent) is left out: its eigenvalue is 0, its vector zero, and
// it sorts last.  w_out [kRitz][kRitz] row-major (column m: the m-th Ritz vector's coefficients), lam descending.
__device__ __forceinline__ void pencil_eigen(double g, double h, double* __restrict__ w_out, double* __restrict__ lam_out,
                                             int32_t* __restrict__ dead_out) {
    const int lane = threadIdx.x & 63, i = lane >> 3, j = lane & 7;
    // unit diagonal
    const double gd = shfl_f64(g, 9 * i), gdj = shfl_f64(g, 9 * j);
    const double si = gd > 0.0 ? 1.0 / sqrt(gd) : 0.0, sj = gdj > 0.0 ? 1.0 / sqrt(gdj) : 0.0;
    g *= si * sj;
    h *= si * sj;
    // forward elimination of G carried out on the identity as well: E = L^-1
    double E = i == j ? 1.0 : 0.0;
    bool dead = false;      // of row i
#pragma unroll
    for (int k = 0; k < kRitz; ++k) {
        const double pivot = shfl_f64(g, 9 * k);
        const double rs = pivot > 1e-13 ? newton_rsqrt<3>(pivot) : 0.0;
        if (i == k && rs == 0.0) dead = true;
        const double lik = shfl_f64(g, 8 * i + k) * rs, ljk = shfl_f64(g, 8 * j + k) * rs;   // L[i][k], L[j][k] (i, j > k)
        const double Ek = shfl_f64(E, 8 * k + j) * rs;                                       // row k of L^-1
        if (i == k) E = Ek;
        if (i > k) E = fma(-lik, Ek, E);
        if (i > k && j > k) g = fma(-lik, ljk, g);
    }
    // S = E H E^T
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < kRitz; ++k) t = fma(shfl_f64(E, 8 * i + k), shfl_f64(h, 8 * k + j), t);
    double S = 0.0;
#pragma unroll
    for (int k = 0; k < kRitz; ++k) S = fma(shfl_f64(t, 8 * i + k), shfl_f64(E, 8 * j + k), S);
    S = 0.5 * (S + shfl_f64(S, 8 * j + i));
    double U = i == j ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 12; ++sweep) {
        const double dii = shfl_f64(S, 9 * i), djj = shfl_f64(S, 9 * j);
        if (!__any(i != j && S * S > 1e-33 * fabs(dii * djj))) break;
        for (int round = 0; round < 7; ++round) {
            // index x < 7 meets (round - x) mod 7, or 7 where that is x itself
            auto partner = [round](int x) {
                if (x == 7) return (4 * round) % 7;
                const int y = (round - x + 7) % 7;
                return y == x ? 7 : y;
            };
            const int ip = partner(i), jp = partner(j);
            const int lo = min(i, ip), hi = max(i, ip);
            const double sll = shfl_f64(S, 9 * lo), shh = shfl_f64(S, 9 * hi), slh = shfl_f64(S, 8 * lo + hi);
            double cs = 1.0, sn = 0.0;
            // tan of the rotation's angle: the smaller root of t^2 + t (shh - sll) / slh - 1.  It only steers the convergence: any t with
            // cs = 1 / sqrt(1 + t^2) to full precision is a rotation.
            const double diff = shh - sll, twice = 2.0 * slh, square = fma(diff, diff, twice * twice);
            if (slh * slh > 1e-34 * fabs(sll * shh) && square > 1e-280) {
                const double t = fabs(twice) * newton_rcp<2>(fabs(diff) + square * newton_rsqrt<2>(square));
                const double tt = diff == 0.0 || (diff > 0.0) == (slh > 0.0) ? t : -t;
                cs = newton_rsqrt<3>(fma(tt, tt, 1.0));
                sn = tt * cs;
            }
            const double sg = i == lo ? -sn : sn;                       // row i <- cs row i + sg row ip
            const double cj = shfl_f64(cs, 8 * j), sgj = shfl_f64(sg, 8 * j);
            const double r = fma(sg, shfl_f64(S, 8 * ip + j), cs * S);
            S = fma(sgj, shfl_f64(r, 8 * i + jp), cj * r);
            U = fma(sgj, shfl_f64(U, 8 * i + jp), cj * U);
        }
    }
    // W = D E^T U, columns in descending order of the eigenvalues
    double W = 0.0;
#pragma unroll
    for (int k = 0; k < kRitz; ++k) W = fma(shfl_f64(E, 8 * k + i), shfl_f64(U, 8 * k + j), W);
    W *= si;
    const int row_dead = dead ? 1 : 0;
    const int col_dead = __shfl(row_dead, 8 * j, 64);
    const double lam = col_dead ? 0.0 : shfl_f64(S, 9 * j);
    if (col_dead) W = 0.0;
    int rank = 0;
#pragma unroll
    for (int k = 0; k < kRitz; ++k) {
        const double lk = shfl_f64(lam, k);                 // lane k: row 0, column k
        const int dk = __shfl(col_dead, k, 64);
        rank += dk != col_dead ? (dk < col_dead) : (lk > lam || (lk == lam && k < j));
    }
    w_out[i * kRitz + rank] = W;
    if (i == 0) { lam_out[rank] = lam; dead_out[rank] = col_dead; }
}

// LDS of a Rayleigh-Ritz step
template <int THREADS>
struct RitzLds {
    double part[THREADS / 64][2][kRitz * kRitz];   // partial sums of G and H per wavefront
    double W[kRitz * kRitz], lam[kRitz];
    double red[THREADS / 64][2];
    int32_t dead[kRitz];
};

// One Rayleigh-Ritz step in one workgroup of THREADS >= d.  Q [d][kRitz] any block, Z = C Q (LDS, row-major).  On return
// Q holds the Ritz vectors, Z the next Chebyshev iterate (C - c) / e Q, and `st` (LDS or global, written by thread 0) what
// comes next.  A dependent column is replaced by a coordinate vector.
template <int THREADS>
__device__ __forceinline__ void ritz_step(double* __restrict__ Q, double* __restrict__ Z, const double* __restrict__ C, int32_t d, int32_t p,
                                          RitzLds<THREADS>& L, RitzState& st) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kWaves = THREADS / 64;
    {
        const int a = lane >> 3, b = lane & 7;
        double g = 0.0, h = 0.0;
        for (int r = wave; r < d; r += kWaves) {
            const double qa = Q[r * kRitz + a];
            g = fma(qa, Q[r * kRitz + b], g);
            h = fma(qa, Z[r * kRitz + b], h);
        }
        L.part[wave][0][lane] = g;
        L.part[wave][1][lane] = h;
    }
    __syncthreads();
    if (wave == 0) {
        double g = 0.0, h = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { g += L.part[w][0][lane]; h += L.part[w][1][lane]; }
        h = 0.5 * (h + shfl_f64(h, 8 * (lane & 7) + (lane >> 3)));
        pencil_eigen(g, h, L.W, L.lam, L.dead);
    }
    __syncthreads();
    double rq[kRitz], rz[kRitz];
    double e0 = 0.0, e1 = 0.0;
    if (tid < d) {
#pragma unroll
        for (int m = 0; m < kRitz; ++m) { rq[m] = 0.0; rz[m] = 0.0; }
#pragma unroll
        for (int a = 0; a < kRitz; ++a) {
            const double qa = Q[tid * kRitz + a], za = Z[tid * kRitz + a];
#pragma unroll
            for (int m = 0; m < kRitz; ++m) {
                rq[m] = fma(qa, L.W[a * kRitz + m], rq[m]);
                rz[m] = fma(za, L.W[a * kRitz + m], rz[m]);
            }
        }
        const double d0 = rz[0] - L.lam[0] * rq[0], d1 = rz[1] - L.lam[1] * rq[1];
        e0 = d0 * d0;
        e1 = d1 * d1;
    }
    for (int w = 32; w > 0; w >>= 1) { e0 += __shfl_xor(e0, w, 64); e1 += __shfl_xor(e1, w, 64); }
    if (lane == 0) { L.red[wave][0] = e0; L.red[wave][1] = e1; }
    __syncthreads();
    if (tid == 0) {
        double s0 = 0.0, s1 = 0.0;
        for (int w = 0; w < kWaves; ++w) { s0 += L.red[w][0]; s1 += L.red[w][1]; }
        const double l0 = L.lam[0];
        const double r0 = l0 > 0.0 ? sqrt(s0) / l0 : 0.0, resid = l0 > 0.0 ? fmax(r0, sqrt(s1) / l0) : 0.0;
        for (int m = 0; m < kRitz; ++m) st.lam[m] = L.lam[m];
        st.resid = resid;
        st.steps += 1;
        // Upper end of the interval: the block's smallest Ritz value.  Inside a cluster of more than kRitz equal eigenvalues
        // that end lies in the cluster and nothing is gained on what is below: after four steps without progress, one step
        // with a lower end.
        double shrink = 1.0;
        if (resid > 0.5 * st.best) {
            if (++st.stall >= 4) { shrink = 0.8; st.stall = 0; }
        } else {
            st.best = resid;
            st.stall = 0;
        }
        // The first direction leaks into the other columns at the level rho of its error; the polynomial amplifies the leak
        // by its value at lam_1.  Held at 1e4 relative to 1 the scaled Gram matrix stays factorable with digits to spare.
        const double rho = fmax(r0, 1e-15), room = 9.2 - log(rho);
        const double b = fmax(shrink * L.lam[p - 1], 2e-4 * rho * l0);
        int deg = kMaxDegree;
        if (b > 0.0) {
            const double x1 = 2.0 * l0 / b - 1.0, x2 = 2.0 * L.lam[p > 1 ? 1 : 0] / b - 1.0;
            if (x1 > 1.0 + 1e-9) deg = min(deg, (int)(room / acosh(x1)));
            if (x2 > 1.0 + 1e-6 && resid > 0.0) deg = min(deg, (int)ceil(log(resid / 1e-13) / acosh(x2)));   // what is left to gain
        }
        st.degree = max(1, deg);
        st.c = 0.5 * b;
        st.e = 0.5 * b;
    }
    __syncthreads();
    if (tid < d) {
        const double c = st.c, inv_e = st.e > 0.0 ? 1.0 / st.e : 0.0;
        const int salt = st.steps * 101;
#pragma unroll
        for (int m = 0; m < kRitz; ++m) {
            if (m < p && L.dead[m]) {   // a fresh direction; its image is a column of C
                const int unit = (m * 37 + salt) % d;
                rq[m] = tid == unit ? 1.0 : 0.0;
                rz[m] = C[(int64_t)tid * d + unit];
            }
            Q[tid * kRitz + m] = rq[m];
            Z[tid * kRitz + m] = (rz[m] - c * rq[m]) * inv_e;
        }
    }
    __syncthreads();
}

// entry x of the start block [d][kRitz]: a fixed pseudo-random number in [-1, 1) (SplitMix64, G. L. Steele, D. Lea and C. H. Flood 2014, of
// the counter x), zero in the columns >= p
__device__ __forceinline__ double start_entry(int x, int32_t p) {
    if (x % kRitz >= p) return 0.0;
    uint64_t h = ((uint64_t)x + 1u) * 0x9E3779B97F4A7C15ull;
    h = (h ^ (h >> 30)) * 0xBF58476D1CE4E5B9ull;
    h = (h ^ (h >> 27)) * 0x94D049BB133111EBull;
    h ^= h >> 31;
    return (double)(h >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

__global__ void __launch_bounds__(256) k_pca_start(double* __restrict__ Q, int32_t d, int32_t p, RitzState* __restrict__ st) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x < d * kRitz) Q[x] = start_entry(x, p);
    if (x == 0) { *st = RitzState{}; st->best = 1e300; }
}

// One 16-row tile of C times a block [d][kRitz] on the float64 matrix cores, by the 16 wavefronts of a workgroup: every
// wavefront multiplies its share of the columns, the partial tiles are added in wavefront order.  Returns the product for
// (row, column) = (tid / kRitz, tid % kRitz) in the threads tid < 16 kRitz.
__device__ __forceinline__ double tile_product(const double* __restrict__ C, const double* __restrict__ Y, int32_t d, int row0,
                                               double (*part)[16 * kRitz]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane >> 4, lc = lane & 15;
    const int row = min(row0 + lc, d - 1);
    constexpr int kSteps = (kMaxDim / 4 + 15) / 16;     // steps of four columns per wavefront, at most
    double a[kSteps], y[kSteps];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
        const int k = 4 * (wave + 16 * s) + lr;
        const bool live = k < d;
        a[s] = live ? C[(int64_t)row * d + k] : 0.0;
        y[s] = live && lc < kRitz ? Y[k * kRitz + lc] : 0.0;
    }
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
        if (4 * (wave + 16 * s) < d) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], y[s], acc, 0, 0, 0);
    if (lc < kRitz) {
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave][(lr + 4 * v) * kRitz + lc] = acc[v];
    }
    __syncthreads();
    double sum = 0.0;
    if (threadIdx.x < 16 * kRitz)
#pragma unroll
        for (int w = 0; w < 16; ++w) sum += part[w][threadIdx.x];
    return sum;
}

// out = C y (prev == nullptr) or the Chebyshev step out = 2 (C y - c y) / e - prev; a workgroup per 16 rows
__global__ void __launch_bounds__(kRitzThreads) k_pca_apply(const double* __restrict__ C, const double* __restrict__ y, const double* __restrict__ prev,
                                                            const RitzState* __restrict__ st, int32_t d, double* __restrict__ out) {
    __shared__ double part[16][16 * kRitz];
    const int row0 = blockIdx.x * 16, x = row0 * kRitz + (int)threadIdx.x;
    const bool live = threadIdx.x < 16 * kRitz && x < d * kRitz;
    // what the last line needs is fetched ahead of the product: three memory latencies less in a kernel made of them
    const double yx = live && prev ? y[x] : 0.0, px = live && prev ? prev[x] : 0.0, c = st->c, e = st->e;
    const double v = tile_product(C, y, d, row0, part);
    if (live) out[x] = prev ? 2.0 * (v - c * yx) / e - px : v;
}

// the Rayleigh-Ritz step on a block in global memory: Q in (the block), out (the Ritz vectors); Z in (C Q), out (the next iterate)
__global__ void __launch_bounds__(kRitzThreads) k_pca_ritz(const double* __restrict__ C, double* __restrict__ Q, double* __restrict__ Z, int32_t d,
                                                           int32_t p, RitzState* __restrict__ st) {
    extern __shared__ double block[];   // Q, Z
    __shared__ RitzLds<kRitzThreads> L;
    __shared__ RitzState s;
    static_assert(kMaxDim <= kRitzThreads && kSmallDim <= kSmallThreads, "one row per thread");
    double *q = block, *z = block + (size_t)d * kRitz;
    for (int x = threadIdx.x; x < d * kRitz; x += kRitzThreads) { q[x] = Q[x]; z[x] = Z[x]; }
    if (threadIdx.x == 0) s = *st;
    __syncthreads();
    ritz_step<kRitzThreads>(q, z, C, d, p, L, s);
    for (int x = threadIdx.x; x < d * kRitz; x += kRitzThreads) { Q[x] = q[x]; Z[x] = z[x]; }
    if (threadIdx.x == 0) *st = s;
}

// The whole iteration for d <= kSmallDim in one workgroup: the block stays in LDS, a wavefront keeps its 16 rows of C in
// registers (STEPS of four columns).  A chain of multiplications by C, each waiting for the one before: all that a wavefront reads of the
// block is on its way before the first matrix instruction, nothing is behind a branch and no division is left in it.
// The 4x4x4 instruction works on four blocks, lane l: row (of A) or column (of B) l % 4 of block l / 4 % 4, k = l / 16; it receives
// row l / 16, column l % 4.  Two blocks of rows and two of columns make 8 x 8 of the product, where half of the 16x16x4 one's
// columns would be idle.  Five steps at 128 columns 289 -> 246 us (270 with the instruction alone), at 96 231 -> 178, four at 50 139 -> 130.
template <int STEPS>
__global__ void __launch_bounds__(kSmallThreads) k_pca_axes_small(const double* __restrict__ C, double* __restrict__ Q, int32_t d, int32_t p,
                                                                  double tol, int32_t max_steps, RitzState* __restrict__ st_out) {
    __shared__ double Y[2][kSmallDim * kRitz];
    __shared__ RitzLds<kSmallThreads> L;
    __shared__ RitzState st;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane >> 4, lc = lane & 15;
    double a[2][STEPS];
    const int row0 = wave * 16, arow = row0 + 4 * (lc >> 3) + (lc & 3), col = lc & 7, drow = row0 + 4 * (lc >> 3) + lr;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int s = 0; s < STEPS; ++s) a[u][s] = arow + 8 * u < d && 4 * s + lr < d ? C[(int64_t)(arow + 8 * u) * d + 4 * s + lr] : 0.0;
    for (int x = tid; x < kSmallDim * kRitz; x += kSmallThreads) {   // rows beyond d stay zero
        Y[0][x] = x < d * kRitz ? start_entry(x, p) : 0.0;
        Y[1][x] = 0.0;
    }
    if (tid == 0) { st = RitzState{}; st.best = 1e300; }
    __syncthreads();
    // Y[to] = C Y[from], or the Chebyshev step with Y[to] holding the iterate before (all threads call)
    double c = 0.0, inv_e = 0.0;
    auto multiply = [&](int from, int to, bool step) {
        if (row0 < d) {
            double y[STEPS], now[2], before[2];
#pragma unroll
            for (int s = 0; s < STEPS; ++s) y[s] = Y[from][(4 * s + lr) * kRitz + col];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                now[u] = Y[from][(drow + 8 * u) * kRitz + col];
                before[u] = Y[to][(drow + 8 * u) * kRitz + col];
            }
            double acc[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
#pragma unroll
                for (int u = 0; u < 2; ++u) acc[u][s & 1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[u][s], y[s], acc[u][s & 1], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const double r = acc[u][0] + acc[u][1];
                Y[to][(drow + 8 * u) * kRitz + col] = step ? 2.0 * (r - c * now[u]) * inv_e - before[u] : r;
            }
        }
        __syncthreads();
    };
    int q = 0;      // Y[q] is the block (later the iterate before), Y[q ^ 1] its image (the newest iterate)
    multiply(q, q ^ 1, false);
    for (int step = 0; step < max_steps; ++step) {
        ritz_step<kSmallThreads>(Y[q], Y[q ^ 1], C, d, p, L, st);
        if (!(st.resid > tol) || step + 1 == max_steps) break;
        const int degree = st.degree;
        c = st.c;
        inv_e = 1.0 / st.e;
        for (int k = 1; k < degree; ++k) { multiply(q ^ 1, q, true); q ^= 1; }
        multiply(q ^ 1, q, false);
        q ^= 1;
    }
    for (int x = tid; x < d * kRitz; x += kSmallThreads) Q[x] = Y[q][x];
    if (tid == 0) *st_out = st;
}

// factor[m] for m = 0, 1: the sign that makes the axis' entry of largest magnitude (the first among equals) positive,
// times std0 / sqrt(lam_1) when std0 > 0.  One wavefront per axis.
__global__ void __launch_bounds__(128) k_pca_orient(const double* __restrict__ Q, int32_t d, const RitzState* __restrict__ st, float std0,
                                                    double* __restrict__ factor) {
    const int m = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double best = -1.0, value = 0.0;
    int at = d;
    for (int r = lane; r < d; r += 64) {
        const double v = Q[r * kRitz + m];
        if (fabs(v) > best) { best = fabs(v); value = v; at = r; }
    }
    for (int w = 32; w > 0; w >>= 1) {
        const double ob = __shfl_xor(best, w, 64), ov = __shfl_xor(value, w, 64);
        const int oa = __shfl_xor(at, w, 64);
        if (ob > best || (ob == best && oa < at)) { best = ob; value = ov; at = oa; }
    }
    if (lane == 0) factor[m] = (value > 0.0 ? 1.0 : -1.0) * (std0 > 0.f ? (double)std0 / sqrt(st->lam[0]) : 1.0);
}

// theta_i = factor * ((x_i - mean) . axis_1, (x_i - mean) . axis_2).  LANES lanes share a row (a power of two, enough for
// one VEC-wide chunk of the row each), 64 / LANES rows side by side in a wavefront, kProjectRows such groups in flight: the
// loop is a stream of X from memory (512 MB at 128 columns: 0.27 ms with four 4-byte loads in flight per lane, 0.134 with eight of 16
// bytes; halving the sums a lane holds at every step of the reduction, 16 exchanges for 80, takes 0.205).
constexpr int kProjectRows = 8;
template <int VEC, int LANES>
__global__ void __launch_bounds__(256) k_pca_project(const float* __restrict__ X, int64_t n, int32_t d, const double* __restrict__ mean,
                                                     const double* __restrict__ Q, const double* __restrict__ factor,
                                                     float* __restrict__ theta) {
    constexpr int kSide = 64 / LANES;                 // rows side by side
    const int lane = threadIdx.x & 63, part = lane % LANES, side = lane / LANES;
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (kSide * kProjectRows) + side;
    double s0[kProjectRows], s1[kProjectRows];
#pragma unroll
    for (int u = 0; u < kProjectRows; ++u) { s0[u] = 0.0; s1[u] = 0.0; }
    for (int col = VEC * part; col < d; col += VEC * LANES) {
        float v[kProjectRows][VEC];
#pragma unroll
        for (int u = 0; u < kProjectRows; ++u) {
            const float* src = X + min(row0 + (int64_t)u * kSide, n - 1) * d + col;
            if (VEC == 4) { const float4 t = *(const float4*)src; v[u][0] = t.x; v[u][1 % VEC] = t.y; v[u][2 % VEC] = t.z; v[u][3 % VEC] = t.w; }
            else v[u][0] = *src;
        }
#pragma unroll
        for (int w = 0; w < VEC; ++w) {
            const double m = mean[col + w], q0 = Q[(col + w) * kRitz], q1 = Q[(col + w) * kRitz + 1];
#pragma unroll
            for (int u = 0; u < kProjectRows; ++u) {
                const double c = (double)v[u][w] - m;
                s0[u] = fma(c, q0, s0[u]);
                s1[u] = fma(c, q1, s1[u]);
            }
        }
    }
    const double f0 = factor[0], f1 = factor[1];
#pragma unroll
    for (int u = 0; u < kProjectRows; ++u) {
        for (int o = LANES / 2; o > 0; o >>= 1) {
            s0[u] += __shfl_xor(s0[u], o, 64);
            s1[u] += __shfl_xor(s1[u], o, 64);
        }
        const int64_t row = row0 + (int64_t)u * kSide;
        if (part == 0 && row < n) { theta[2 * row] = (float)(s0[u] * f0); theta[2 * row + 1] = (float)(s1[u] * f1); }
    }
}

}  // namespace nomad_pca
