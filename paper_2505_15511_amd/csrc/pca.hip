// libnomad: the PCA initialisation behind the C ABI of include/nomad.h (host side).
#include <hip/hip_runtime.h>

#include <cmath>

#include "host_util.h"
#include "nomad.h"
#include "pca_kernels.h"
#include "rows.h"

using namespace nomad_pca;

#pragma GCC visibility push(default)
extern "C" int nomad_pca_init(const float* X, int64_t n, int32_t d, float std0, float* theta_out, double* stats, int mem, int32_t device,
                              void* stream) {
    if (!X || !theta_out || (mem != NOMAD_HOST && mem != NOMAD_DEVICE)) return NOMAD_E_INVALID_ARG;
    if (n < 2 || d < 2 || d > kMaxDim || device < 0 || !(std0 == std0)) return NOMAD_E_INVALID_ARG;
    if (n >= ((int64_t)1 << 31) - 256) return NOMAD_E_TOO_LARGE;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return NOMAD_E_HIP;
    KTRY(hipSetDevice(device));
    hipStream_t st = (hipStream_t)stream;
    Buffers buf(st);
    const float* dX = X;
    float* dTheta = theta_out;
    if (mem == NOMAD_HOST) {
        float *x = nullptr, *t = nullptr;
        KTRY(buf.alloc(&x, (size_t)n * d));
        KTRY(buf.alloc(&t, (size_t)n * 2));
        KTRY(hipMemcpyAsync(x, X, sizeof(float) * (size_t)n * d, hipMemcpyHostToDevice, st));
        dX = x; dTheta = t;
    }
    const int32_t p = std::min<int32_t>(kRitz, d);
    // covariance about a shift, and the mean with it: as many (tile pair, slab) wavefronts as the chip holds at once, two per SIMD
    // (every one is a long chain of matrix instructions, so none is left over for a second round); slabs of at least 256 rows
    const int32_t nb = (d + kColBlock - 1) / kColBlock, n_off = nb * (nb - 1) / 2, n_pairs = nb + n_off;
    const auto cut = [&](double want, int32_t& count, int64_t& rows) {
        const int64_t slabs64 = std::max<int64_t>(1, std::min<int64_t>((int64_t)want, (n + 255) / 256));
        rows = (((n + slabs64 - 1) / slabs64) + 3) / 4 * 4;
        count = (int32_t)((n + rows - 1) / rows);
    };
    CovSlabs slabs;
    const double off_slabs = 2048.0 / (n_off + kDiagonalShare * nb);
    cut(off_slabs, slabs.off, slabs.off_rows);
    cut(kDiagonalShare * off_slabs, slabs.diag, slabs.diag_rows);
    const size_t tiles = (size_t)nb * slabs.diag + (size_t)n_off * slabs.off;
    double *cov_partial = nullptr, *Cm = nullptr, *sums = nullptr, *shift = nullptr, *delta = nullptr, *mean = nullptr;
    KTRY(buf.alloc(&cov_partial, tiles * kColBlock * kColBlock));
    KTRY(buf.alloc(&Cm, (size_t)d * d));
    KTRY(buf.alloc(&sums, (size_t)slabs.diag * d));
    KTRY(buf.alloc(&shift, (size_t)d)); KTRY(buf.alloc(&delta, (size_t)d)); KTRY(buf.alloc(&mean, (size_t)d));
    hipLaunchKernelGGL(k_pca_shift, dim3(blocks_of(d, 64)), dim3(64 * kMeanWaves), 0, st, dX, n, d, shift);
    hipLaunchKernelGGL(k_pca_cov, dim3((uint32_t)tiles), dim3(64), 0, st, dX, n, d, (const double*)shift, slabs, cov_partial, sums);
    hipLaunchKernelGGL(k_pca_mean, dim3(blocks_of(d, 64)), dim3(64 * kMeanWaves), 0, st, (const double*)sums, slabs.diag, d, n, (const double*)shift, delta, mean);
    hipLaunchKernelGGL(k_pca_cov_reduce, dim3(blocks_of((int64_t)n_pairs * kColBlock * kColBlock, kReduceEntries)), dim3(256), 0, st,
                       (const double*)cov_partial, slabs, d, n, (const double*)delta, Cm);
    // leading eigenvectors: subspace iteration from a fixed pseudo-random block
    double *Q = nullptr, *Z = nullptr, *factor = nullptr;
    RitzState* state = nullptr;
    KTRY(buf.alloc(&Q, (size_t)d * kRitz));
    KTRY(buf.alloc(&Z, (size_t)d * kRitz));
    KTRY(buf.alloc(&state, 1));
    KTRY(buf.alloc(&factor, 2));
    RitzState hstate{};
    const double tol = 1e-12;
    const int max_steps = 2000;
    if (d <= kSmallDim) {
        const auto kernel = d <= 32 ? k_pca_axes_small<8> : d <= 64 ? k_pca_axes_small<16> : d <= 96 ? k_pca_axes_small<24> : k_pca_axes_small<kSmallDim / 4>;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kSmallThreads), 0, st, (const double*)Cm, Q, d, p, tol, max_steps, state);
        KTRY(hipMemcpyAsync(&hstate, state, sizeof(hstate), hipMemcpyDeviceToHost, st));
        KTRY(hipStreamSynchronize(st));
    } else {
        double* Zp = nullptr;
        KTRY(buf.alloc(&Zp, (size_t)d * kRitz));
        const size_t lds = (size_t)2 * d * kRitz * sizeof(double);
        KTRY(hipFuncSetAttribute((const void*)k_pca_ritz, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(k_pca_start, dim3(blocks_of((int64_t)d * kRitz, 256)), dim3(256), 0, st, Q, d, p, state);
        auto apply = [&](const double* y, const double* prev, double* out) {
            hipLaunchKernelGGL(k_pca_apply, dim3(blocks_of(d, 16)), dim3(kRitzThreads), 0, st, (const double*)Cm, y, prev, (const RitzState*)state, d, out);
        };
        double *block = Q, *image = Z, *spare = Zp;
        apply(block, nullptr, image);
        while (true) {
            hipLaunchKernelGGL(k_pca_ritz, dim3(1), dim3(kRitzThreads), lds, st, (const double*)Cm, block, image, d, p, state);
            KTRY(hipMemcpyAsync(&hstate, state, sizeof(hstate), hipMemcpyDeviceToHost, st));
            KTRY(hipStreamSynchronize(st));
            if (!(hstate.resid > tol) || hstate.steps >= max_steps) break;
            double *before = block, *now = image;   // T_0 and T_1 of the block
            for (int k = 1; k < hstate.degree; ++k) {
                apply(now, before, spare);
                double* t = before; before = now; now = spare; spare = t;
            }
            apply(now, nullptr, before);
            block = now; image = before;
        }
        Q = block;
    }
    KTRY(hipGetLastError());
    if (std0 > 0.f && !(hstate.lam[0] > 0.0)) return NOMAD_E_INVALID_ARG;   // no variance to scale
    // scores
    hipLaunchKernelGGL(k_pca_orient, dim3(1), dim3(128), 0, st, (const double*)Q, d, (const RitzState*)state, std0, factor);
    const auto project = [&](auto kernel, int lanes) {
        hipLaunchKernelGGL(kernel, dim3(blocks_of(n, 4 * (64 / lanes) * kProjectRows)), dim3(256), 0, st, dX, n, d, (const double*)mean, (const double*)Q,
                           (const double*)factor, dTheta);
    };
    if (rows_by_16(dX, d)) {
        if (d <= 32) project(k_pca_project<4, 8>, 8);
        else if (d <= 64) project(k_pca_project<4, 16>, 16);
        else if (d <= 128) project(k_pca_project<4, 32>, 32);
        else project(k_pca_project<4, 64>, 64);
    } else if (d <= 16) project(k_pca_project<1, 16>, 16);
    else project(k_pca_project<1, 64>, 64);
    KTRY(hipGetLastError());
    if (mem == NOMAD_HOST) KTRY(hipMemcpyAsync(theta_out, dTheta, sizeof(float) * (size_t)n * 2, hipMemcpyDeviceToHost, st));
    KTRY(hipStreamSynchronize(st));
    if (stats) {
        stats[0] = hstate.lam[0];
        stats[1] = hstate.lam[1];
        stats[2] = hstate.resid;
        stats[3] = (double)hstate.steps;
    }
    return NOMAD_OK;
}
#pragma GCC visibility pop
