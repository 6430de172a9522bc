// libnomad: how many wavefronts share a workgroup of the neighbour filter inside clusters, and which slices of one set share their distances, plain C++
// (a test compiles it with the host compiler).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

namespace nomad_knn {

constexpr int64_t kFilterUnits = 256;   // compute units, one workgroup of the filter at a time each
constexpr int kFilterLists = 8;         // XCDs: workgroups go to them in turn, and each works through a list of its own (filter_blocks)

// The lists are poured full in turn, an eighth of the work each: the end of list x, and the list that a workgroup goes to when `done` of the work is in the lists already
// and the one before went to `list`.  (Whole numbers below 2^53: exact.)
inline double filter_list_end(int list, double total) { return list + 1 < kFilterLists ? (double)(list + 1) * total / kFilterLists : 1e300; }
inline int filter_list(int list, double done, double total) {
    while (done >= filter_list_end(list, total)) ++list;
    return list;
}

// The groups with tiles, longest first: by counting, unless one is far longer than there are groups.
inline std::vector<uint32_t> longest_first(const std::vector<uint32_t>& tstart) {
    const size_t groups = tstart.size() - 1;
    const auto tiles = [&](size_t g) { return tstart[g + 1] - tstart[g]; };
    uint32_t most = 0;
    for (size_t g = 0; g < groups; ++g) most = std::max(most, tiles(g));
    std::vector<uint32_t> order;
    if (most > 16 * groups) {
        for (size_t g = 0; g < groups; ++g)
            if (tiles(g)) order.push_back((uint32_t)g);
        std::sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) { return tiles(a) > tiles(b); });
        return order;
    }
    std::vector<uint32_t> at((size_t)most + 2, 0u);   // at[c]: groups of more than c tiles, and then where the next of c goes
    for (size_t g = 0; g < groups; ++g)
        if (tiles(g)) ++at[tiles(g) - 1];
    for (uint32_t c = most; c-- > 0;) at[c] += at[c + 1];
    order.resize(at[0]);
    for (size_t g = 0; g < groups; ++g)
        if (tiles(g)) order[at[tiles(g)]++] = (uint32_t)g;
    return order;
}

// How long UNITS compute units are at work on workgroups that are added longest first: one that begins a round has the mean of those before it ahead of it.
template <int64_t UNITS>
struct FilterList {
    int64_t count = 0;
    double before = 0.0, span = 0.0;
    void add(uint32_t c, int64_t m) {   // m of them, c tiles each
        const int64_t round = (count + m - 1) / UNITS * UNITS;   // the last that begins a round; those before it among the m have less ahead
        if (round >= count) span = std::max(span, (before + (double)(round - count) * (double)c) / (double)UNITS + (double)c);
        before += (double)m * (double)c;
        count += m;
    }
};

// How long the filter is at work over groups of tstart[g + 1] - tstart[g] tiles, in tiles of candidates, `waves` tiles of queries to a workgroup: the mean of the longest list's
// span and of the whole chip's as if it were one list.  (Few long clusters can leave one XCD with a round more than the others.  Neither says enough alone: 68,277 x 76 in 12 clusters twelve over eight wavefronts 1.00 by the chip, 0.82 by the lists and 1.16 measured, 95,776 x 59 in 11 0.51, 0.97 and 0.89.)
// By groups, not by workgroups, for the device waits meanwhile: 1,000,000 x 128 in 256 clusters, host 270 -> 5 us, the call 5.35 -> 5.00 ms (5.18 and 5.01 without the rule).
inline double filter_span(const std::vector<uint32_t>& tstart, const std::vector<uint32_t>& order, int waves) {
    const size_t groups = tstart.size() - 1;
    const auto tiles = [&](size_t g) { return tstart[g + 1] - tstart[g]; };
    const auto workgroups = [&](size_t g) { return (int64_t)((tiles(g) + (uint32_t)waves - 1u) / (uint32_t)waves); };
    double total = 0.0, done = 0.0;
    for (const uint32_t g : order) total += (double)tiles(g) * (double)workgroups(g);
    // the lists that the groups' workgroups go to: piece[at[g]] .. of group g
    struct Piece { int32_t list; uint32_t count; };
    std::vector<Piece> piece(groups + 2 * kFilterLists);   // (one a group, and one more where a list ends inside a group)
    std::vector<uint32_t> at(groups + 1);
    uint32_t pieces = 0;
    int list = 0;
    double end = filter_list_end(0, total);
    for (size_t g = 0; g < groups; ++g) {
        at[g] = pieces;
        const double c = (double)tiles(g);
        for (int64_t left = workgroups(g); left > 0;) {
            if (done >= end) {
                list = filter_list(list, done, total);
                end = filter_list_end(list, total);
            }
            const int64_t here = done + c * (double)(left - 1) < end ? left : (int64_t)std::ceil((end - done) / c);   // those that begin before the list's end
            piece[pieces++] = Piece{list, (uint32_t)here};
            done += c * (double)here;
            left -= here;
        }
    }
    at[groups] = pieces;
    FilterList<kFilterUnits> chip;
    FilterList<kFilterUnits / kFilterLists> lists[kFilterLists];
    for (size_t i = 0; i < order.size();) {   // groups of one length at a time
        const uint32_t c = tiles(order[i]);
        int64_t of[kFilterLists] = {}, all = 0;
        for (; i < order.size() && tiles(order[i]) == c; ++i)
            for (uint32_t x = at[order[i]]; x < at[order[i] + 1]; ++x) of[piece[x].list] += piece[x].count;
        for (int l = 0; l < kFilterLists; ++l)
            if (of[l]) {
                lists[l].add(c, of[l]);
                all += of[l];
            }
        chip.add(c, all);
    }
    double longest = 0.0;
    for (const auto& l : lists) longest = std::max(longest, l.span);
    return 0.5 * (longest + chip.span);
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
    if (eight < kMany) {
        const std::vector<uint32_t> order = longest_first(tstart);
        all8 = filter_span(tstart, order, 8);
        all = filter_span(tstart, order, most);
    }
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
