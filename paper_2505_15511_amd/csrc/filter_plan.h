// libnomad: how many wavefronts share a workgroup of the neighbour filter inside clusters, and which slices of one set share their distances, plain C++
// (a test compiles it with the host compiler).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace nomad_knn {

constexpr int64_t kFilterUnits = 256;   // compute units, one workgroup of the filter at a time each
constexpr int kFilterLists = 8;         // XCDs: workgroups go to them in turn, and each works through a list of its own (filter_blocks)

// the list that a workgroup goes to when `done` of the work is in the lists already
inline int filter_list(double done, double total) { return total > 0.0 ? std::min(kFilterLists - 1, (int)(done / total * kFilterLists)) : 0; }

// How long `units` compute units are at work on workgroups of these lengths, longest first: one that begins a round has the mean of those before it ahead of it.
inline double list_span(std::vector<uint32_t>& list, int64_t units) {
    std::sort(list.begin(), list.end(), [](uint32_t a, uint32_t b) { return a > b; });
    double span = 0.0, before = 0.0;
    for (size_t i = 0; i < list.size(); ++i) {
        if ((int64_t)i % units == 0) span = std::max(span, before / (double)units + (double)list[i]);
        before += (double)list[i];
    }
    return span;
}

// How long the filter is at work over groups of tstart[g + 1] - tstart[g] tiles, in tiles of candidates, `waves` tiles of queries to a workgroup: the mean of the longest list's
// span and of the whole chip's as if it were one list.  (Few long clusters can leave one XCD with a round more than the others.  Neither says enough alone: 68,277 x 76 in 12 clusters twelve over eight wavefronts 1.00 by the chip, 0.82 by the lists and 1.16 measured, 95,776 x 59 in 11 0.51, 0.97 and 0.89.)
inline double filter_span(const std::vector<uint32_t>& tstart, int waves) {
    double total = 0.0, done = 0.0, longest = 0.0;
    std::vector<uint32_t> all, lists[kFilterLists];
    for (size_t g = 0; g + 1 < tstart.size(); ++g) {
        const uint32_t c = tstart[g + 1] - tstart[g], count = (c + (uint32_t)waves - 1u) / (uint32_t)waves;
        all.insert(all.end(), count, c);
        total += (double)c * (double)count;
    }
    for (const uint32_t c : all) {
        lists[filter_list(done, total)].push_back(c);
        done += (double)c;
    }
    for (auto& l : lists) longest = std::max(longest, list_span(l, kFilterUnits / kFilterLists));
    return 0.5 * (longest + list_span(all, kFilterUnits));
}

// Eight wavefronts share a staged tile, or `most` (twelve or sixteen, as the registers allow).  These are faster by themselves where a workgroup's wavefronts have work, for
// three or four wavefronts a SIMD hide what two wait for; but workgroups are fewer then and longer, one of sixteen 1.4 to 1.5 times as long as one of eight, one of twelve 1.1 to 1.25.
// The line is where the span is nine tenths.  Calls, `most` over eight, by span over span (330 sets of 16,400 to 300,000 rows of 4 to 384 columns in 5 to 1,400 clusters, equal
// and of very different sizes, half of them up to 60): below 0.6 0.86 in the mean, 0.6 to 0.8 0.93, 0.8 to 0.9 0.98 (0.90 to 1.12), 0.9 to 0.95 1.02, 0.95 to 0.99 1.08, 1 1.10
// (0.97 to 1.24).  By this line 0.2 % above the better of the two in the mean, 12 % at most (220 other sets: 0.6 and 8 %); always eight 4 and 39 %, always `most` 5 and 24 %; by the span of the
// chip as one list 0.4 and 29 % (46,542 x 180 in eleven clusters, k = 21, 1.18 ms where twelve take 1.01).
inline int filter_waves(const std::vector<uint32_t>& tstart, int most) {
    if (most <= 8) return 8;
    constexpr int64_t kMany = 16 * kFilterUnits;   // workgroups from which rounds don't count
    int64_t eight = 0;
    double all8 = 0.0, all = 0.0;
    for (size_t g = 0; g + 1 < tstart.size(); ++g) {
        const uint32_t c = tstart[g + 1] - tstart[g];
        eight += (c + 7u) / 8u;
        all8 += (double)c * (double)((c + 7u) / 8u);
        all += (double)c * (double)((c + (uint32_t)most - 1u) / (uint32_t)most);
    }
    if (eight < kMany) { all8 = filter_span(tstart, 8); all = filter_span(tstart, most); }
    return 10.0 * all < 9.0 * all8 ? most : 8;
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
