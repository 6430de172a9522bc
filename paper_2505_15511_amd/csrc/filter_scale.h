// libnomad: scales and error bound of the nearest-neighbour filter, plain C++ (the kernels use them on the device, a test
// compiles them with the host compiler).  Squared norms are passed as the bit patterns of non-negative float32 numbers, which
// order like the numbers; infinity and NaN of either sign come after every finite one.
#pragma once
#include <math.h>
#include <stdint.h>
#include <string.h>

#if defined(__HIP__)
#define NOMAD_BOTH __host__ __device__ __forceinline__
#else
#define NOMAD_BOTH inline
#endif

namespace nomad_knn {

// x of M = f 2^x, 1/2 <= f < 1 (0 for M = 0)
NOMAD_BOTH int knn_exponent(uint32_t bits) {
    float M;
    memcpy(&M, &bits, sizeof(M));
    int x = 0;
    (void)frexpf(M, &x);
    return x;
}
// Scale of a group's rows: the power of two 2^e that brings |x'| <= sqrt(M) to at most 2^14.
NOMAD_BOTH int knn_scale_exponent(uint32_t max_bits) {
    const int e = 14 - ((knn_exponent(max_bits) + 1) >> 1);
    return e < -60 ? -60 : e > 60 ? 60 : e;
}
// Whether every key of a group is a finite number, scaled as the filter multiplies it and as it passes it on.  Both sides'
// largest centred squared norms are at most 2^120 (keys are at most three times that), and |c'|^2 / 2 in units of both scales
// is below 2^119: the scaled products are at most 2^28, but a side of tiny rows next to a side of huge ones scales the latter's
// norms by the former's factor.  Groups that are not usable (a sentinel of 1e20 among the rows, rows that are no numbers) are
// left to the exact path as a whole.
NOMAD_BOTH bool knn_filter_usable(uint32_t q_bits, uint32_t c_bits) {
    constexpr uint32_t kLargest = (uint32_t)(127 + 120) << 23;
    return q_bits <= kLargest && c_bits <= kLargest && knn_exponent(c_bits) + knn_scale_exponent(q_bits) + knn_scale_exponent(c_bits) <= 120;
}
// Bound on |filter key - exact key| for rows of d values whose centred squared norms are at most M, u = 2^-24:
//   products     hi hi + hi lo + lo hi leaves out lo lo and what lo was rounded by: 3 2^-22 |q||c|; float16 numbers below
//                2^-14 taken as zero: 2^-13 of a scaled row element, 2^-28 sqrt(d) |q||c| (or, where the scale is at its
//                limit, 2^-72 sqrt(d M)); doubled in the key
//   sums         |c|^2 / 2 and d products, each addition rounded by at most 2 u of the sum of magnitudes, at most 3/2 M
//                (whatever the order inside a matrix instruction), doubled in the key: 6 (d + 1) u M; the two small
//                products' sums are 2^-10 of that
//   norm, final combination, centring in float32: (d + 8) u M + 8 u M
//   underflow    a square is a multiple of 2^-149 and zero below 2^-150: norms miss up to d 2^-150 each, and a side whose M
//                came out as zero is multiplied as zero: at most 4 d 2^-150 < 1e-40 in the key (next to a larger side:
//                2 sqrt(d) 2^-75 sqrt(M), inside the products' term)
// chunk > 0: the large products are summed `chunk` columns at a time, the first chunk on top of |c|^2 / 2, and the chunks' sums
// added up; the norm is kNormLanes sums side by side, each of at most 4 ceil(d / 64) squares, added pairwise.  Then
//   sums         inside a chunk `chunk` additions of at most 2 u of the chunk's own magnitudes, which add up to 3/2 M at most over
//                the chunks (Cauchy-Schwarz); a rounding of u 3/2 M a chunk and one for the small products; doubled in the key:
//                6 chunk u M + 3 (d / chunk + 2) u M; the two small products' own sums are 2^-10 of 8 d u M
//   norm         4 ceil(d / 64) + 4 additions: (d / 16 + 10) u M
// which for 768 columns in chunks of 64 is a tenth of the bound for one sum, for 128 columns half of it.
constexpr int kNormLanes = 16;   // lanes that share a row's norm
NOMAD_BOTH double knn_filter_eps(int32_t d, double M, int32_t chunk = 0) {
    const double units = chunk > 0 ? 6.0 * (double)(chunk + 1) + 3.0 * ((double)d / (double)chunk + 2.0) + (double)d / (double)kNormLanes + 10.0 + (double)d / 64.0 + 64.0
                                   : 7.0 * (double)(d + 4) + 64.0;
    return units * 5.9604644775390625e-08 * M * 1.01 + 1e-12 * M + 1e-20 * sqrt(M) + 1e-40;
}

}  // namespace nomad_knn
