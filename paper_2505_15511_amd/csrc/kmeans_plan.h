// libnomad: which steps of Lloyd's iterations take one launch, plain C++ (a test compiles it with the host compiler).
// Times in this file: per iteration, one launch less the launches it stands for, one MI355X, Gaussian mixtures.
#pragma once
#include <stdint.h>

#include "filter_scale.h"

namespace nomad_knn {

// The M step in one launch (k_mean_small) instead of a sort by label, its scans and the sums.  It saves 10 to 30 us where
//   clusters are short and points few, because a workgroup reads all labels and adds its centroid's rows one after the other, 1.4 ns a label
//   and 16 a row: n + 12 n / K up to 20,000 (d = 4 to 116: 1,040 points, K = 2 -19 us; 3,000, K = 2 -4 to 0; 4,800, K = 6 -7; 7,200, K = 6 -1 to +2;
//   9,000, K = 10 -1; 10,000, K = 10 +2; 11,200, K = 16 -6 to -1; 15,000, K = 10 +17; 16,000, K = 16 +6 to +11, K = 64 -4 to -8; d = 768 10 to 20 us less);
//   the workgroups, one a centroid and 64 columns, are not many rounds of the chip: 1,024 (4,000 points, K = 512, d = 128 -23, K = 256, d = 300
//   +2, K = 512, d = 768 +36; 2,000 points, K = 128, d = 768 -2);
//   the labels, which every workgroup reads, are not much: 2^23 of them (16,000 points, d <= 64, K = 512 -17 to -21, K = 1,024 +2 to +6; K = 256, d = 128
//   +2, d = 300 +33; K = 64, d = 300 -14, d = 768 +4; 16,000 points, K = 2,000, d = 768 +900: 6.8 ms a call for 2.0).
constexpr int64_t kSmallMeanPoints = 16384;   // (the workgroup's list of them is 16-bit, in LDS)
inline bool mean_in_one_launch(int64_t n, int64_t K, int64_t d) {
    const int64_t workgroups = K * ((d + 63) / 64);
    return n <= kSmallMeanPoints && n * K + 12 * n <= 20000 * K && workgroups <= 1024 && n * workgroups <= ((int64_t)1 << 23);
}

// Positions of a partial sum in the parallel M step: 512, fewer where that leaves compute units idle (100,003 x 768, 196 workgroups: 98 us), but not
// where clusters are long: k_mean_combine adds a cluster's partial sums one after the other, which short rows hide less of.  128 / 256 positions
// against 512, us, d = 64: 20,000 points, K = 32 -3 / -2, K = 8 0 / 0, K = 2 +3 / +2; 50,000, K = 16 0 / -2, K = 4 +6 / 0; 100,000, K = 32 0 / -3, K = 8 +7 / 0,
// K = 128 -6 / -5, K = 2 +24 / +6; 300,000, K = 64 +7 / +2, K = 4 +72 / +25 (and d = 16: 960 us a call of five iterations for 887); d = 768: 20,000, K = 8 -16 / -11, K = 2 -8 / -7;
// 50,000, K = 8 -23 / -21, K = 2 -2 / -9; 100,000, K = 64 -9 / -14, K = 8 +16 / 0, K = 4 +10 / -3, K = 2 +26 / +6.
inline int32_t mean_span(int64_t n, int64_t K, int64_t d) {
    if (n < (d < 256 ? 98304 : 65536) && n <= (16 + d / 32) * 128 * K) return 128;
    if (n < 512 * 1024 && n <= (32 + d / 12) * 256 * K) return 256;
    return 512;
}

// Clearing, norms, packing and the copy of the centroids in one launch (k_kmeans_prepare), whose every workgroup reads all K rows, 64
// at a time: -6 to -13 us up to K = 128, -1 to -8 at 512, about 0 at 640, +4 at 1,024, +15 at 2,048, +38 at 4,096 (d = 2 to 64), +83 at 8,192.
constexpr int64_t kPrepareValues = 65536;     // (128 x 768 -4, 256 x 300 -3: there by a margin)
inline bool prepare_in_one_launch(int64_t K, int64_t d) { return K <= 640 && K * d <= kPrepareValues; }

// What the filter leaves open goes to the exact path at once, over all K centroids, instead of to the candidates' refinement first: a
// launch less.  Up to 16,384 points -2 to -10 us, wide rows to -40; from K = 1,024 on -24 to +55.
inline bool open_points_are_few(int64_t n, int64_t K) { return n <= 16384 && K <= 768; }

// Tiles of points whose open points a wavefront of k_assign_refine takes: few, for it takes them 16 at a time (8 in 16-row tiles), a chain of d float64 additions each; but a
// wavefront's start is not free either.  Calls of five steps on rows without structure, 2 / 4 / 8 / 16 tiles, ms: 1,250 tiles (20,000 x 768) 1.07 / 1.15 / 1.27 / 1.50,
// 6,251 (100,003 x 768) 2.64 / 2.66 / 2.75 / 3.18, 9,375 (300,000 x 64) 0.98 / 0.95 / 0.94 / 0.94, 31,250 (1,000,000 x 128) 3.89 / 3.84 / 3.81 / 3.75; one tile 4 % slower than two.
constexpr int kRefineTiles = 16;      // at most (a wavefront's queue in LDS)
inline int32_t refine_tiles(int64_t n_tiles) {
    const int64_t tiles = (n_tiles + 2047) / 2048;
    return (int32_t)(tiles < 2 ? 2 : tiles < kRefineTiles ? tiles : kRefineTiles);
}

// Which wavefronts count, for the host, what the large products leave open of their tile of points: one in kOpenSample.  The workgroups' points lie in eight
// lists, an eighth of all points each, in turn (filter_blocks): tile t of list x is counted where t comes to a place among 64 that differs from list to list and
// from 64 tiles to the next, so that rows in any order of their own, classes one after the other or a period, are met as often as they are there.  (One workgroup in
// 64 is always the first list's: 1,000,000 x 128 with an eighth in clusters, which come first, and the rest without structure, 13.1 ms a call of six steps, now 4.7.)
constexpr uint32_t kOpenSample = 64;
NOMAD_BOTH bool open_is_counted(uint32_t workgroup, uint32_t wave) {
    const uint32_t list = workgroup % 8u, tile = workgroup / 8u * 8u + wave;   // (eight wavefronts a workgroup)
    return tile % kOpenSample == (9u * list + 37u * (tile / kOpenSample)) % kOpenSample;
}

// Whether the filter may do without the small products where the large ones decide, in steps after one that has left few points open: a step saves
// 3e-6 ns of filter a product (n K d of them) and pays for the points that are open then, counting them costs a few us a call.  Calls of five steps, never / always
// alone, ms: n K d = 2.7e8 (65,536, K = 64, d = 64) 0.588 / 0.597, 8.2e8 (100,003, K = 128, d = 64) 0.614 / 0.627, 1.1e9 (66,000, K = 256, d = 64) 0.608 / 0.606, 1.7e9
// (35,000, K = 64, d = 768) 1.072 / 1.033, 3.2e9 (50,000, K = 500, d = 128) 0.827 / 0.793, 1.2e10 (300,000, K = 128, d = 300) 2.21 / 1.82, 7.7e10 (50,000, K = 2,000,
// d = 768) 3.83 / 3.56; short rows of many points, whose filter the additional operand of a query is as much as: 1,000,000, K = 16, d = 16 0.996 / 1.083.  Fewer than
// eight wavefronts a workgroup (n_tiles tiles of points) have no such instance.
// Rows that are not read 16 bytes at a time (by16): what is open, however little, waits for chains of d loads (100,003 x 231, K = 128: filter 39 -> 20 us a step, but refinement
// 22 -> 33 and exact path 21 -> 54), which a step saves from about n K = 2^26 on.  Calls of ten steps, never / with them, ms, by n K: 1.3e7 (100,003 x 231, 128) 1.92 / 2.27,
// (100,003 x 129, 128) 1.40 / 1.51, 1.5e7 (60,001 x 255, 256) 1.78 / 2.02, 2.6e7 (200,000 x 127, 128) 1.85 / 1.92, 3.0e7 (150,000 x 230, 200) 2.09 / 2.07, 3.8e7
// (300,000 x 98, 128) 1.80 / 1.81, 1.3e8 (500,000 x 67, 256) 2.58 / 2.37.
inline bool products_may_be_alone(int64_t n, int64_t K, int64_t d, int64_t n_tiles, int64_t steps, bool by16) {
    return (by16 || n * K >= (int64_t)1 << 26) && steps > 1 && n_tiles >= 1024 && K * d >= 8192 && n * K * d >= (int64_t)1 << 30 && !open_points_are_few(n, K);
}
// The share of the points, at most, that a step may leave open for the next to do so: what is open costs a row of each of its candidates, and of all centroids where
// these don't decide, which is as much as the step saves at about K d / 2^20: 300,000, K = 128, d = 64, saved 9 us, paid at a share of 0.016 3, 0.027 18, 0.045 49;
// 1,000,000, K = 256, d = 128, saved 90, paid at 0.014 20, 0.034 73.
inline bool products_alone(int64_t open, int64_t n, int64_t K, int64_t d) {
    const int64_t products = K * d * (d > 256 ? 3 : 1);      // (16-row tiles: 2.5 to 3 times as long a product)
    const int64_t share = products < 65536 ? (((int64_t)1 << 20) + products - 1) / products : 16;
    return open * share < n;
}

}  // namespace nomad_knn
