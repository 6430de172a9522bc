// libnomad: how many wavefronts share a workgroup of the neighbour filter inside clusters, and which slices of one set share their distances, plain C++
// (a test compiles it with the host compiler).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace nomad_knn {

constexpr int64_t kFilterUnits = 256;   // compute units, one workgroup of the filter at a time each

// How long the filter is at work over groups of hist[c] groups of c tiles each, in tiles of candidates, `waves` tiles of queries to a workgroup: longest groups first, and a
// workgroup that begins a round of the chip has the mean of those before it ahead of it.
inline double filter_span(const std::vector<uint32_t>& hist, int waves) {
    double span = 0.0, before = 0.0;   // candidates' tiles of the workgroups so far
    int64_t at = 0;                    // workgroups so far
    for (size_t c = hist.size(); c-- > 1;) {
        if (hist[c] == 0u) continue;
        const int64_t count = (int64_t)hist[c] * (int64_t)((c + (size_t)waves - 1) / (size_t)waves);
        const int64_t last = (at + count - 1) / kFilterUnits * kFilterUnits;   // the last of them that begins a round
        if (last >= at) span = std::max(span, (before + (double)(last - at) * (double)c) / (double)kFilterUnits + (double)c);
        before += (double)count * (double)c;
        at += count;
    }
    return span;
}

// Eight wavefronts share a staged tile, or `most` (twelve or sixteen, as the registers allow).  These are faster by themselves where a workgroup's wavefronts have work, for
// three or four wavefronts a SIMD hide what two wait for; but workgroups are fewer then and longer, one of sixteen 1.4 to 1.5 times as long as one of eight, one of twelve 1.1 to 1.25.
// The line is where the span is six sevenths.  Calls, `most` over eight, by span over span (420 sets of 33,000 to 400,000 rows of 16 to 300 columns, clusters of 200
// to 4,000, equal and Dirichlet): up to 0.6 0.74 to 0.94; 0.65 to 0.75 0.83 to 1.01; 0.8 to 0.85 0.78 to 1.03; 0.86 to 0.96 1.03 to 1.16; 1, where the longest cluster or a
// last round decides, 0.91 to 1.28 (1.06 to 1.13 in the mean).  By this line 0.3 % above the better of the two in the mean, 10 % at most; always eight 4 and 32 %, always `most` 5 and 28 %.
inline int filter_waves(const std::vector<uint32_t>& tstart, int most) {
    if (most <= 8) return 8;
    constexpr int64_t kMany = 16 * kFilterUnits;   // workgroups from which rounds don't count
    int64_t eight = 0;
    double all8 = 0.0, all = 0.0;
    uint32_t longest = 0u;
    for (size_t g = 0; g + 1 < tstart.size(); ++g) {
        const uint32_t c = tstart[g + 1] - tstart[g];
        eight += (c + 7u) / 8u;
        all8 += (double)c * (double)((c + 7u) / 8u);
        all += (double)c * (double)((c + (uint32_t)most - 1u) / (uint32_t)most);
        longest = std::max(longest, c);
    }
    if (eight >= kMany) return 7.0 * all < 6.0 * all8 ? most : 8;
    std::vector<uint32_t> hist((size_t)longest + 1, 0u);
    for (size_t g = 0; g + 1 < tstart.size(); ++g) ++hist[tstart[g + 1] - tstart[g]];
    return 7.0 * filter_span(hist, most) < 6.0 * filter_span(hist, 8) ? most : 8;
}

// Whether slices of one set tell each other how near their candidates are: a wavefront does so some ten times over 4,000 candidates, twenty over 16,000, forty over 166,000, each
// time reading 16 bytes a slice and lane (four lanes a query in 16-row tiles, two in 32-row ones), and what it saves goes with the candidates.  Calls, shared over not,
// by slices x candidates: 2 x 5,000 1.07, 4 x 9,661 1.04, 6 x 7,750 1.00, 8 x 14,650 0.93, 8 x 57,546 0.79; 17 x 4,201 1.07, 17 x 11,593 1.07, 17 x 22,513 0.99, 12 x 21,890 0.98,
// 12 x 36,285 0.94; 25 x 12,000 1.05, 21 x 47,620 0.96; 16-row tiles 2 x 13,007 1.04, 6 x 4,349 1.18, 12 x 15,901 1.06, 6 x 16,668 0.94; long lists in 32-row tiles, whose hits
// take longer, 4 x 4,523 1.03, 6 x 7,750 1.00, 8 x 12,500 0.95.
inline bool slices_share(int64_t slices, int64_t candidates, int tile, bool long_list) {
    constexpr int64_t kMost = 32;
    return slices > 1 && slices <= kMost && candidates >= (long_list && tile == 32 ? 8192 : 14336) && candidates * tile >= 1280 * 32 * slices;
}

}  // namespace nomad_knn
