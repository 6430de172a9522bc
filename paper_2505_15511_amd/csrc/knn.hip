// libnomad: the upstream index (K-Means, in-cluster exact nearest neighbours) and the quality measures behind the C ABI of
// include/nomad.h (host side).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

#include "filter_plan.h"
#include "host_util.h"
#include "kmeans_plan.h"
#include "knn_filter.h"
#include "knn_kernels.h"
#include "metrics_kernels.h"
#include "nomad.h"

using namespace nomad_knn;
using namespace nomad_metrics;

namespace {

void launch_norms(hipStream_t st, const float* X, int64_t n, int32_t d, const int32_t* members, const int32_t* group_of, const float* centre, float* norm,
                  uint32_t* max_bits) {
    hipLaunchKernelGGL(k_knn_norms, dim3((uint32_t)((n + norm_block_rows(n) - 1) / norm_block_rows(n))), dim3(256), 0, st, X, n, d, members, group_of, centre, norm,
                       max_bits, (int32_t)norm_batches(n));
}

// One side of the filter, packed: tiles per group (host and device), the packed rows, and the launch that fills them.
struct PackedSide {
    int tile = 32, steps = 1;
    int32_t groups = 0;
    uint32_t n_tiles = 0;
    std::vector<uint32_t> tstart;          // [groups + 1]
    const uint32_t *d_start = nullptr, *d_tstart = nullptr;
    uint4* data = nullptr;
    float* norm = nullptr;

    void plan(const std::vector<uint32_t>& start, int32_t d, int32_t list_len) {
        tile = knn_tile(d, list_len);
        steps = knn_steps(d, tile);
        groups = (int32_t)start.size() - 1;
        tstart.assign(start.size(), 0u);
        for (int32_t g = 0; g < groups; ++g) tstart[g + 1] = tstart[g] + (start[g + 1] - start[g] + (uint32_t)tile - 1) / (uint32_t)tile;
        n_tiles = tstart[groups];
    }
    int alloc(Buffers& buf, bool with_norm) {
        KTRY(buf.alloc(&data, ((size_t)n_tiles + kMaxStageTiles) * knn_tile_units(steps)));   // a stage may read past the last tile
        if (with_norm) KTRY(buf.alloc(&norm, ((size_t)n_tiles + kMaxStageTiles) * tile));
        return NOMAD_OK;
    }
    void fill(hipStream_t st, const float* X, int32_t d, const int32_t* members, const float* centre, const uint32_t* max_bits,
              const uint32_t* other_bits, const float* row_norm) {
        if (n_tiles)
            hipLaunchKernelGGL(k_knn_pack, dim3(n_tiles), dim3(256), 0, st, X, d, members, d_start, d_tstart, groups, centre, max_bits,
                               other_bits, row_norm, tile,
                               steps, data, norm);
    }
    KnnPacked view(const uint32_t* max_bits) const { return KnnPacked{data, norm, d_tstart, max_bits}; }
};

// The filter's work list: `waves` query tiles of one group per workgroup.  Workgroups go to the 8 XCDs in turn, and each XCD
// has an L2 of its own: the work is poured into eight lists of equal cost, group after group, so that the workgroups that
// stream a group's candidates share an L2 (a group is cut only where a list is full).  Inside a list the groups with the
// most candidates come first: a workgroup's time goes with its group's candidates, and what starts last should be short.
// Entries without work (cluster -1) fill the shorter lists up.
std::vector<KnnBlock> filter_blocks(const PackedSide& Q, const PackedSide& C, int waves) {
    const auto cost_of = [&](int32_t g) { return (double)(C.tstart[g + 1] - C.tstart[g]); };
    double total = 0.0;
    for (int32_t g = 0; g < Q.groups; ++g) total += cost_of(g) * (double)((Q.tstart[g + 1] - Q.tstart[g] + (uint32_t)waves - 1) / (uint32_t)waves);
    std::vector<KnnBlock> lists[kFilterLists];
    double done = 0.0;
    int list = 0;
    for (int32_t g = 0; g < Q.groups; ++g)
        for (uint32_t t = 0; t < Q.tstart[g + 1] - Q.tstart[g]; t += (uint32_t)waves) {
            lists[list = filter_list(list, done, total)].push_back(KnnBlock{g, (int32_t)t});
            done += cost_of(g);
        }
    size_t longest = 0;
    for (auto& l : lists) {
        std::stable_sort(l.begin(), l.end(), [&](const KnnBlock& a, const KnnBlock& b) { return cost_of(a.cluster) > cost_of(b.cluster); });
        longest = std::max(longest, l.size());
    }
    std::vector<KnnBlock> blocks(longest * kFilterLists, KnnBlock{-1, 0});
    for (int x = 0; x < kFilterLists; ++x)
        for (size_t i = 0; i < lists[x].size(); ++i) blocks[i * kFilterLists + (size_t)x] = lists[x][i];
    return blocks;
}

constexpr uint32_t kLoopGrid = 512;   // workgroups of the kernels whose work list is counted on the device

// The k nearest candidates of every query inside its group (filter, refinement, exact fallback).  `cand` [n_q * (k + kPad)],
// `tau` [n_q], `flagged` [n_q], `n_flagged` [1] (zero) are work space.
int nearest_in_groups(hipStream_t st, Buffers& buf, const KnnSets& P, const KnnBlock* blocks, uint32_t n_blocks, int waves, int32_t k, int32_t* cand, float* keys, float* tau,
                      int32_t* flagged, uint32_t* n_flagged, int32_t* out) {
    const int32_t list_len = k + kPad;
    const dim3 grid((uint32_t)std::min<int64_t>(P.n_q, kLoopGrid));
    ExactParts parts{};
    KTRY(buf.alloc(&parts.D, (size_t)grid.x * k)); KTRY(buf.alloc(&parts.P, (size_t)grid.x * k)); KTRY(buf.alloc(&parts.done, (size_t)grid.x));
    KTRY(hipMemsetAsync(parts.done, 0, sizeof(uint32_t) * (size_t)grid.x, st));
    KTRY(launch_knn_filter(st, n_blocks, waves, P, blocks, list_len, cand, keys, tau, KnnAssign{}));
    if (list_len <= 16)
        hipLaunchKernelGGL(k_knn_refine<16>, dim3(blocks_of(P.n_q, 16)), dim3(256), 0, st, P, cand, keys, tau, k, list_len, out, flagged, n_flagged);
    else if (list_len <= 32)
        hipLaunchKernelGGL(k_knn_refine<32>, dim3(blocks_of(P.n_q, 8)), dim3(256), 0, st, P, cand, keys, tau, k, list_len, out, flagged, n_flagged);
    else
        hipLaunchKernelGGL(k_knn_refine<64>, dim3(blocks_of(P.n_q, 4)), dim3(256), 0, st, P, cand, keys, tau, k, list_len, out, flagged, n_flagged);
    if (k <= 16) hipLaunchKernelGGL((k_knn_exact<16, 1024>), grid, dim3(1024), 0, st, P, flagged, (const uint32_t*)n_flagged, k, out, parts);
    else hipLaunchKernelGGL((k_knn_exact<kMaxK, 512>), grid, dim3(512), 0, st, P, flagged, (const uint32_t*)n_flagged, k, out, parts);
    KTRY(hipGetLastError());
    return NOMAD_OK;
}

// The nearest candidate of every query (one group).  Work space: cand [n_q * 128 / tile], tau, flagged [n_q], open [tiles of queries],
// n_flagged (zero).  few: what the filter leaves open goes to the exact path at once (kmeans_plan.h).  Query positions are query rows here.
int nearest_one(hipStream_t st, const KnnSets& P, int tile, const KnnBlock* blocks, uint32_t n_blocks, int waves, bool few, int32_t* cand, float* tau,
                uint32_t* open, int32_t* flagged, uint32_t* n_flagged, int32_t* out) {
    KTRY(launch_knn_filter(st, n_blocks, waves, P, blocks, 1, cand, nullptr, tau, few ? KnnAssign{out, flagged, n_flagged, nullptr} : KnnAssign{out, nullptr, nullptr, open}));
    if (!few) {
        const int64_t n_tiles = (P.n_q + tile - 1) / tile;
        const int32_t tiles = refine_tiles(n_tiles);
        hipLaunchKernelGGL(k_assign_refine, dim3(blocks_of(n_tiles, 4 * tiles)), dim3(256), 0, st, P, (const uint32_t*)open, n_tiles, tile, tiles, (const int32_t*)cand,
                           (const float*)tau, 128 / tile, out, flagged, n_flagged);
    }
    hipLaunchKernelGGL((k_knn_exact<1, 256>), dim3((uint32_t)std::min<int64_t>(P.n_q, kLoopGrid)), dim3(256), 0, st, P, (const int32_t*)flagged,
                       (const uint32_t*)n_flagged, 1, out, ExactParts{});
    KTRY(hipGetLastError());
    return NOMAD_OK;
}

constexpr int32_t kZeroWords = 6;   // counters of an iteration, then the centroids' largest norm

// The M step of Lloyd's iteration: the points sorted by label with a stable radix sort (ascending point order inside a
// cluster), then float64 sums in that order per (centroid, column); a label without points leaves its centroid as it is.
// sort() and means() only enqueue.
struct MeanStep {
    int64_t n = 0;
    int32_t K = 0, d = 0;
    int passes = 1;                 // radix passes of 8 bits that cover the labels 0..K-1
    uint32_t n_blocks = 0;          // workgroups of a sort pass
    bool parallel = false;          // clusters of 128 points and more on average: column sums in parallel (k_mean_partials)
    uint32_t *lstart = nullptr, *hist = nullptr, *tile_total = nullptr, *list = nullptr;
    MeanPartial* partial = nullptr;
    int32_t span = 0;               // positions of a partial sum
    uint32_t n_tiles = 0;           // tiles of the scan over the 256 n_blocks digit counters
    int32_t* stamp_of = nullptr;    // [K] sort with prev that last saw the cluster change
    int32_t stamp = 0;
    ChangedClusters clusters{nullptr, 0, 0};   // of the last sort
    int32_t *keys[2] = {nullptr, nullptr}, *ids[2] = {nullptr, nullptr};   // a pass reads one pair of arrays and writes the other
    const int32_t *sorted_keys = nullptr, *sorted_ids = nullptr;

    bool small = false;             // everything in one launch (k_mean_small)

    int init(Buffers& buf, int64_t n_, int32_t K_, int32_t d_) {
        n = n_; K = K_; d = d_;
        small = mean_in_one_launch(n, K, d);
        if (small) return NOMAD_OK;
        int bits = 1;
        while (((int64_t)1 << bits) < K) ++bits;
        passes = (bits + 7) / 8;
        n_blocks = blocks_of(n, kSortSpan);
        parallel = n >= (int64_t)128 * K;
        span = mean_span(n, K, d);
        KTRY(buf.alloc(&lstart, (size_t)K + 1));
        KTRY(buf.alloc(&stamp_of, (size_t)K));
        n_tiles = (uint32_t)(((size_t)256 * n_blocks + kScanTile - 1) / kScanTile);
        KTRY(buf.alloc(&hist, (size_t)256 * n_blocks));
        KTRY(buf.alloc(&tile_total, (size_t)n_tiles));
        for (int x = 0; x < (passes > 1 ? 2 : 1); ++x) { KTRY(buf.alloc(&keys[x], (size_t)n)); KTRY(buf.alloc(&ids[x], (size_t)n)); }
        if (parallel) {
            KTRY(buf.alloc(&partial, ((size_t)blocks_of(n, span) + (size_t)K) * d));
            KTRY(buf.alloc(&list, (size_t)K * d));
        }
        return NOMAD_OK;
    }
    // labels [n] in 0..K-1 (on the device); with prev the labels that differ are counted (*changed: zero), and means() leaves the centroids of
    // clusters that have not changed alone: they are the means of prev's.  host: is handed that count, and *open_count in the high half
    int sort(hipStream_t st, const int32_t* labels, const int32_t* prev = nullptr, unsigned long long* changed = nullptr, HostWord* host = nullptr,
             const uint32_t* open_count = nullptr) {
        const int32_t* kin = labels;
        const int32_t* vin = nullptr;   // first pass: the point at position i is i
        int out = 0;
        if (!prev) stamp = 0;
        const ChangedClusters stamps{stamp_of, prev ? ++stamp : 0, K};
        clusters = prev ? stamps : ChangedClusters{nullptr, 0, 0};
        for (int p = 0; p < passes; ++p) {
            const bool report = p == 0 && host;
            hipLaunchKernelGGL(k_sort_count, dim3(n_blocks), dim3(256), 0, st, kin, n, 8 * p, n_blocks, hist,
                               p == 0 ? prev : (const int32_t*)nullptr, changed, report ? host->word() : (unsigned long long*)nullptr, open_count, stamps,
                               p == 0 && !prev ? K : 0);
            if (report) KTRY(host->record(st));
            hipLaunchKernelGGL(k_sort_scan_tiles, dim3(n_tiles), dim3(256), 0, st, hist, (uint64_t)256 * n_blocks, tile_total);
            hipLaunchKernelGGL(k_sort_scan, dim3(1), dim3(1024), 0, st, tile_total, (uint64_t)n_tiles);
            hipLaunchKernelGGL(k_sort_scatter, dim3(n_blocks), dim3(256), 0, st, kin, vin, n, 8 * p, n_blocks, (const uint32_t*)hist,
                               (const uint32_t*)tile_total, keys[out], ids[out], K, passes == 1 ? lstart : (uint32_t*)nullptr);
            kin = keys[out]; vin = ids[out];
            out ^= 1;
        }
        sorted_keys = kin;
        sorted_ids = vin;
        if (passes > 1) hipLaunchKernelGGL(k_label_starts, dim3(blocks_of(n + 1, 256)), dim3(256), 0, st, sorted_keys, n, K, lstart);
        return NOMAD_OK;
    }
    // small sets: dC [K * d] in and out, and the labels that differ from prev's; *changed: zero
    int small_means(hipStream_t st, const float* dX, const int32_t* labels, const int32_t* prev, float* dC, unsigned long long* changed, unsigned long long* changed_host) {
        hipLaunchKernelGGL(k_mean_small, dim3((uint32_t)K, blocks_of(d, 64)), dim3(256), sizeof(uint16_t) * (size_t)n, st, dX, (int32_t)n, d, labels, prev, dC, changed, changed_host);
        KTRY(hipGetLastError());
        return NOMAD_OK;
    }
    // after sort: dC [K * d] in and out; *n_list is zero
    int means(hipStream_t st, const float* dX, float* dC, uint32_t* n_list) {
        const uint32_t entries = blocks_of((int64_t)K * d, 256);
        if (!parallel) {
            hipLaunchKernelGGL(k_kmeans_update, dim3(entries), dim3(256), 0, st, dX, d, sorted_ids, (const uint32_t*)lstart, K, clusters, dC);
        } else {
            const auto sums = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(blocks_of(n, span)), dim3(256), 0, st, dX, n, d, sorted_keys, sorted_ids, (const uint32_t*)lstart, span, clusters, partial);
            };
            // columns per lane: no lane idle before 16-byte loads, as far as rows are aligned for them
            if (d > 128 && rows_by_16(dX, d)) sums(k_mean_partials<4>);
            else if (d % 2 == 0 && d > 64 && ((uintptr_t)dX & 7) == 0) sums(k_mean_partials<2>);
            else sums(k_mean_partials<1>);
            hipLaunchKernelGGL(k_mean_combine, dim3(entries), dim3(256), 0, st, (const MeanPartial*)partial, d, (const uint32_t*)lstart, K, span, clusters, dC, list, n_list);
            hipLaunchKernelGGL(k_mean_ordered, dim3((uint32_t)std::min<int64_t>(2048, (int64_t)K * d)), dim3(256), 0, st, dX, d, sorted_ids,
                               (const uint32_t*)lstart, (const uint32_t*)list, (const uint32_t*)n_list, dC);
        }
        KTRY(hipGetLastError());
        return NOMAD_OK;
    }
};

}  // namespace

#pragma GCC visibility push(default)
extern "C" int nomad_knn_in_clusters(const float* X, int64_t n, int32_t d, const int32_t* cluster_of, int32_t n_clusters, int32_t k,
                                     int32_t* out_nbrs, int mem, int32_t device, void* stream, int64_t* stats) {
    if (!X || !cluster_of || !out_nbrs || (mem != NOMAD_HOST && mem != NOMAD_DEVICE)) return NOMAD_E_INVALID_ARG;
    if (n < 1 || d < 1 || d > NOMAD_KNN_MAX_DIM || n_clusters < 1 || k < 1 || k > NOMAD_KNN_MAX_K || device < 0) return NOMAD_E_INVALID_ARG;
    if (n >= ((int64_t)1 << 31) - 256) return NOMAD_E_TOO_LARGE;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return NOMAD_E_HIP;
    KTRY(hipSetDevice(device));
    hipStream_t st = (hipStream_t)stream;
    Buffers buf(st);
    const int32_t R = n_clusters;
    const int32_t list_len = k + kPad;

    // inputs on the device
    const float* dX = X;
    const int32_t* dC = cluster_of;
    int32_t* dOut = out_nbrs;
    if (mem == NOMAD_HOST) {
        float* x = nullptr;
        int32_t *c = nullptr, *o = nullptr;
        KTRY(buf.alloc(&x, (size_t)n * d));
        KTRY(buf.alloc(&c, (size_t)n));
        KTRY(buf.alloc(&o, (size_t)n * k));
        KTRY(hipMemcpyAsync(x, X, sizeof(float) * (size_t)n * d, hipMemcpyHostToDevice, st));
        KTRY(hipMemcpyAsync(c, cluster_of, sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, st));
        dX = x; dC = c; dOut = o;
    }

    // members grouped by cluster
    uint32_t *counts = nullptr, *cursor = nullptr, *max_norm = nullptr, *n_flagged = nullptr;
    int32_t *members = nullptr, *cand = nullptr, *flagged = nullptr;
    float *norm = nullptr, *keys = nullptr, *tau = nullptr, *centre = nullptr;
    int* bad = nullptr;
    // counters that start at zero: counts, cursor, max_norm, centre, bad, n_flagged
    uint8_t* zeroed = nullptr;
    const size_t zero_words = ((size_t)3 * R + 2 + 3) / 4 * 4;   // ahead of the centres, whose rows are read 16 bytes at a time
    const size_t zero_bytes = sizeof(uint32_t) * (zero_words + (size_t)R * d);
    KTRY(buf.alloc(&zeroed, zero_bytes));
    KTRY(hipMemsetAsync(zeroed, 0, zero_bytes, st));
    counts = (uint32_t*)zeroed; cursor = counts + R; max_norm = cursor + R; bad = (int*)(max_norm + R); n_flagged = (uint32_t*)(bad + 1);
    centre = (float*)zeroed + zero_words;
    KTRY(buf.alloc(&members, (size_t)n));
    KTRY(buf.alloc(&norm, (size_t)n));
    KTRY(buf.alloc(&tau, (size_t)n));
    KTRY(buf.alloc(&cand, (size_t)n * list_len)); KTRY(buf.alloc(&keys, (size_t)n * list_len));
    KTRY(buf.alloc(&flagged, (size_t)n));
    hipLaunchKernelGGL(k_knn_count, dim3(blocks_of(n, kCountSpan)), dim3(256), 0, st, dC, n, R, counts, bad);
    std::vector<uint32_t> hcounts((size_t)3 * R + 1), hstart((size_t)R + 1, 0);   // counts, two arrays of no interest, bad
    KTRY(hipMemcpyAsync(hcounts.data(), counts, sizeof(uint32_t) * hcounts.size(), hipMemcpyDeviceToHost, st));
    KTRY(hipStreamSynchronize(st));
    if (hcounts[(size_t)3 * R]) return NOMAD_E_BAD_GRAPH;   // a cluster id outside 0..n_clusters-1
    const int32_t slab_rows = centroid_rows(n);
    std::vector<KnnBlock> hslabs;
    for (int32_t r = 0; r < R; ++r) {
        hstart[r + 1] = hstart[r] + hcounts[r];
        for (uint32_t q0 = 0; q0 < hcounts[r]; q0 += (uint32_t)slab_rows) hslabs.push_back(KnnBlock{r, (int32_t)q0});
    }
    PackedSide side;
    side.plan(hstart, d, list_len);
    const int eight = knn_filter_waves(side.tile, side.n_tiles);
    const int waves = eight == 8 ? filter_waves(side.tstart, knn_most_waves(side.tile, side.steps, knn_list_class(side.tile, list_len))) : eight;
    const std::vector<KnnBlock> hblocks = filter_blocks(side, side, waves);
    HostArrays up;
    const size_t at_start = up.add(hstart), at_tstart = up.add(side.tstart), at_blocks = up.add(hblocks), at_slabs = up.add(hslabs);
    KTRY(up.upload(buf, st));
    const uint32_t* start = up.at<uint32_t>(at_start);
    const KnnBlock *blocks = up.at<KnnBlock>(at_blocks), *slabs = up.at<KnnBlock>(at_slabs);
    side.d_start = start;
    side.d_tstart = up.at<uint32_t>(at_tstart);
    if (int rc = side.alloc(buf, true)) return rc;
    hipLaunchKernelGGL(k_knn_group, dim3(blocks_of(n, kGroupSpan)), dim3(256), 0, st, dC, n, R, start, cursor, members);
    hipLaunchKernelGGL(k_knn_centroid_sums, dim3((uint32_t)hslabs.size()), dim3(256), 0, st, dX, d, members, start, slabs, slab_rows, centre);
    hipLaunchKernelGGL(k_knn_centroid_finish, dim3(blocks_of((int64_t)R * d, 256)), dim3(256), 0, st, centre, start, R, d);
    const bool ordered = knn_ordered(n, d, R, list_len);   // the order of the rows inside a cluster, and the norms with it
    if (ordered) {
        uint32_t* cells = nullptr;      // [2][R][kCells] counts, cursors
        uint8_t* cell_of = nullptr;
        int32_t* placed = nullptr;
        KTRY(buf.alloc(&cells, (size_t)2 * R * kCells));
        KTRY(buf.alloc(&cell_of, (size_t)n));
        KTRY(buf.alloc(&placed, (size_t)n));
        KTRY(hipMemsetAsync(cells, 0, sizeof(uint32_t) * (size_t)2 * R * kCells, st));
        const size_t lds = sizeof(float) * (size_t)(kCells + 1) * ((d + 3) / 4 * 4);
        hipLaunchKernelGGL(k_knn_cells, dim3((uint32_t)hslabs.size()), dim3(256), lds, st, dX, d, (const int32_t*)members, start, slabs, slab_rows,
                           (const float*)centre, norm, max_norm, cell_of, cells);
        hipLaunchKernelGGL(k_knn_place, dim3((uint32_t)hslabs.size()), dim3(256), 0, st, (const int32_t*)members, (const uint8_t*)cell_of, start, slabs, slab_rows,
                           (const uint32_t*)cells, cells + (size_t)R * kCells, placed);
        members = placed;
    } else {
        launch_norms(st, dX, n, d, members, dC, centre, norm, max_norm);
    }
    side.fill(st, dX, d, members, centre, max_norm, max_norm, norm);

    // filter on the matrix cores, float64 refinement, exact fallback
    KnnSets P{};
    P.XQ = dX; P.XC = dX; P.qmembers = members; P.cmembers = members; P.qstart = start; P.cstart = start;
    P.Q = side.view(max_norm); P.C = P.Q; P.centre = centre; P.group_of_q = dC; P.n_q = n; P.n_c = n; P.d = d; P.same_set = 1; P.ordered = ordered; P.chunk = knn_chunk_columns(d, list_len);
    int rc = nearest_in_groups(st, buf, P, blocks, (uint32_t)hblocks.size(), waves, k, cand, keys, tau, flagged, n_flagged, dOut);
    if (rc) return rc;
    uint32_t hflag = 0;
    KTRY(hipMemcpyAsync(&hflag, n_flagged, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    if (mem == NOMAD_HOST) KTRY(hipMemcpyAsync(out_nbrs, dOut, sizeof(int32_t) * (size_t)n * k, hipMemcpyDeviceToHost, st));
    KTRY(hipStreamSynchronize(st));
    if (stats) {
        stats[0] = (int64_t)hflag;
        int64_t pairs = 0;
        for (int32_t r = 0; r < R; ++r) pairs += (int64_t)hcounts[r] * (int64_t)hcounts[r];
        stats[1] = pairs;
    }
    return NOMAD_OK;
}

extern "C" int nomad_kmeans_lloyd(const float* X, int64_t n, int32_t d, int32_t K, float* centroids, int32_t max_iters, int32_t* labels,
                                  int32_t* iters_out, double* inertia_out, int mem, int32_t device, void* stream) {
    if (!X || !centroids || !labels || (mem != NOMAD_HOST && mem != NOMAD_DEVICE)) return NOMAD_E_INVALID_ARG;
    if (n < 1 || d < 1 || d > NOMAD_KNN_MAX_DIM || K < 1 || K > n || max_iters < 1 || device < 0) return NOMAD_E_INVALID_ARG;
    if (n >= ((int64_t)1 << 31) - 256) return NOMAD_E_TOO_LARGE;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return NOMAD_E_HIP;
    KTRY(hipSetDevice(device));
    hipStream_t st = (hipStream_t)stream;
    Buffers buf(st);
    const float* dX = X;
    float* dC = centroids;
    int32_t* dLab = labels;
    if (mem == NOMAD_HOST) {
        float *x = nullptr, *c = nullptr;
        int32_t* l = nullptr;
        KTRY(buf.alloc(&x, (size_t)n * d));
        KTRY(buf.alloc(&c, (size_t)K * d));
        KTRY(buf.alloc(&l, (size_t)n));
        KTRY(hipMemcpyAsync(x, X, sizeof(float) * (size_t)n * d, hipMemcpyHostToDevice, st));
        KTRY(hipMemcpyAsync(c, centroids, sizeof(float) * (size_t)K * d, hipMemcpyHostToDevice, st));
        dX = x; dC = c; dLab = l;
    }
    // work space
    uint32_t *max_pts = nullptr, *zeros = nullptr;
    uint32_t* open = nullptr;
    int32_t *new_lab = nullptr, *cand = nullptr, *flagged = nullptr;
    float *cnorm = nullptr, *xnorm = nullptr, *tau = nullptr, *centre = nullptr, *c_used = nullptr;
    double* inertia = nullptr;
    const std::vector<uint32_t> hq = {0u, (uint32_t)n}, hc = {0u, (uint32_t)K};
    PackedSide points, cents;
    points.plan(hq, d, 1);
    cents.plan(hc, d, 1);
    KTRY(buf.alloc(&max_pts, 1)); KTRY(buf.alloc(&zeros, kZeroWords));
    KTRY(buf.alloc(&new_lab, (size_t)n)); KTRY(buf.alloc(&cand, (size_t)n * (128 / points.tile))); KTRY(buf.alloc(&open, (size_t)points.n_tiles)); KTRY(buf.alloc(&flagged, (size_t)n));
    KTRY(buf.alloc(&cnorm, (size_t)K)); KTRY(buf.alloc(&tau, (size_t)n)); KTRY(buf.alloc(&centre, (size_t)d)); KTRY(buf.alloc(&c_used, (size_t)K * d));
    KTRY(buf.alloc(&inertia, 1));
    // what every iteration starts from zero: labels changed, the exact path's queries, those the large products leave open (of a sample),
    // columns to add in order; and the largest centred |c|^2
    unsigned long long* changed = (unsigned long long*)zeros;   // (and the workgroups that have counted theirs)
    uint32_t *n_flagged = zeros + 2, *open_count = zeros + 3, *n_list = zeros + 4, *max_cen = zeros + 5;
    const int waves = knn_filter_waves(points.tile, points.n_tiles);
    const std::vector<KnnBlock> hblocks = filter_blocks(points, cents, waves);
    const int32_t slab_rows = centroid_rows(n);
    std::vector<KnnBlock> hslabs;
    for (int64_t q0 = 0; q0 < n; q0 += slab_rows) hslabs.push_back(KnnBlock{0, (int32_t)q0});
    HostArrays up;
    const size_t at_q = up.add(hq), at_c = up.add(hc), at_qt = up.add(points.tstart), at_ct = up.add(cents.tstart), at_blocks = up.add(hblocks),
                 at_slabs = up.add(hslabs);
    KTRY(up.upload(buf, st));
    const uint32_t *qstart = up.at<uint32_t>(at_q), *cstart = up.at<uint32_t>(at_c);
    const KnnBlock *blocks = up.at<KnnBlock>(at_blocks), *slabs = up.at<KnnBlock>(at_slabs);
    points.d_start = qstart; points.d_tstart = up.at<uint32_t>(at_qt);
    cents.d_start = cstart; cents.d_tstart = up.at<uint32_t>(at_ct);
    if (int rc = points.alloc(buf, false)) return rc;
    if (int rc = cents.alloc(buf, true)) return rc;
    // both sides are centred on the mean of the points; the largest centred |x|^2 of the points, once
    KTRY(hipMemsetAsync(centre, 0, sizeof(float) * (size_t)d, st));
    KTRY(hipMemsetAsync(max_pts, 0, sizeof(uint32_t), st));
    hipLaunchKernelGGL(k_knn_centroid_sums, dim3((uint32_t)hslabs.size()), dim3(256), 0, st, dX, d, (const int32_t*)nullptr, qstart, slabs, slab_rows, centre);
    hipLaunchKernelGGL(k_knn_centroid_finish, dim3(blocks_of(d, 256)), dim3(256), 0, st, centre, qstart, 1, d);
    const bool few = open_points_are_few(n, K), may_be_alone = products_may_be_alone(n, K, d, points.n_tiles, max_iters, rows_by_16(dX, d) && rows_by_16(dC, d));
    if (may_be_alone) KTRY(buf.alloc(&xnorm, (size_t)n));
    launch_norms(st, dX, n, d, nullptr, nullptr, centre, xnorm, max_pts);
    points.fill(st, dX, d, nullptr, centre, max_pts, nullptr, nullptr);
    MeanStep m_step;
    {
        int rc = m_step.init(buf, n, K, d);
        if (rc) return rc;
    }

    KnnSets P{};
    P.XQ = dX; P.XC = dC; P.qmembers = nullptr; P.cmembers = nullptr; P.qstart = qstart; P.cstart = cstart;
    P.Q = points.view(max_pts); P.C = cents.view(max_cen); P.centre = centre; P.group_of_q = nullptr; P.n_q = n; P.n_c = K; P.d = d; P.same_set = 0; P.chunk = knn_chunk_columns(d, 1);
    // Labels go back and forth between two arrays; the centroids of the last E step are kept for the inertia.
    int32_t *cur = new_lab, *prev = dLab;
    HostWord hchanged[2];
    for (auto& h : hchanged) KTRY(h.take());
    const bool prepare = prepare_in_one_launch(K, d);
    P.q_norm = xnorm; P.open_count = may_be_alone ? open_count : nullptr;
    int32_t it = 0;
    while (it < max_iters) {
        // E step: the nearest centroid of every point, exactly
        if (prepare) {
            hipLaunchKernelGGL(k_kmeans_prepare, dim3(cents.n_tiles), dim3(1024), 0, st, (const float*)dC, K, d, (const float*)centre, (const uint32_t*)max_pts,
                               cents.tile, cents.steps, cents.data, cents.norm, c_used, zeros, kZeroWords - 1, max_cen);
        } else {
            KTRY(hipMemsetAsync(zeros, 0, kZeroWords * sizeof(uint32_t), st));
            launch_norms(st, dC, K, d, nullptr, nullptr, centre, cnorm, max_cen);
            cents.fill(st, dC, d, nullptr, centre, max_cen, max_pts, cnorm);
            KTRY(hipMemcpyAsync(c_used, dC, sizeof(float) * (size_t)K * d, hipMemcpyDeviceToDevice, st));
        }
        int rc = nearest_one(st, P, points.tile, blocks, (uint32_t)hblocks.size(), waves, few, cand, tau, open, flagged, n_flagged, cur);
        if (rc) return rc;
        ++it;
        const int32_t* before = it > 1 ? prev : nullptr;
        if (m_step.small) {
            // The host runs an iteration ahead: what it has enqueued by the time it learns that nothing moved gives the same centroids
            // and labels again.
            HostWord& h = hchanged[it & 1];
            if ((rc = m_step.small_means(st, dX, cur, before, dC, changed, before ? h.word() : nullptr))) return rc;
            if (before) KTRY(h.record(st));
            std::swap(cur, prev);
            if (it > 2) {
                HostWord& last = hchanged[(it - 1) & 1];
                KTRY(last.wait());
                if (last.value() == 0) { --it; break; }
            }
        } else {
            const bool wait = before || may_be_alone;
            if ((rc = m_step.sort(st, cur, before, changed, wait ? &hchanged[0] : nullptr, P.open_count))) return rc;
            if (before) {   // the device sorts while the host waits for the count; wasted only once, when nothing has changed
                KTRY(hchanged[0].wait());
                if ((uint32_t)hchanged[0].value() == 0) break;   // nothing moved: the centroids are the means of these labels already
            }
            if ((rc = m_step.means(st, dX, dC, n_list))) return rc;
            if (may_be_alone) {
                if (!before) KTRY(hchanged[0].wait());           // (the means are on their way)
                P.alone = products_alone((int64_t)(hchanged[0].value() >> 32) * kOpenSample, n, K, d);
            }
            std::swap(cur, prev);
        }
    }
    // (prev holds the last labels: after a break the two arrays are equal)
    if (prev != dLab) KTRY(hipMemcpyAsync(dLab, prev, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToDevice, st));
    // inertia of the labels against the centroids they were computed from
    double hinertia = 0.0;
    KTRY(hipMemsetAsync(inertia, 0, sizeof(double), st));
    hipLaunchKernelGGL(k_kmeans_inertia, dim3(std::min<uint32_t>(kInertiaGrid, blocks_of(n, kInertiaRows))), dim3(1024), 0, st, dX, (const float*)c_used, d, (const int32_t*)dLab, n, inertia);
    KTRY(hipMemcpyAsync(&hinertia, inertia, sizeof(double), hipMemcpyDeviceToHost, st));
    KTRY(hipGetLastError());
    if (mem == NOMAD_HOST) {
        KTRY(hipMemcpyAsync(centroids, dC, sizeof(float) * (size_t)K * d, hipMemcpyDeviceToHost, st));
        KTRY(hipMemcpyAsync(labels, dLab, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, st));
    }
    KTRY(hipStreamSynchronize(st));
    if (iters_out) *iters_out = it;
    if (inertia_out) *inertia_out = hinertia;
    return NOMAD_OK;
}
extern "C" int nomad_kmeans_lsh_init(const float* X, int64_t n, int32_t d, int32_t K, const float* planes, const int32_t* anchors,
                                     int32_t n_planes, float* centroids_out, int32_t* buckets_out, int mem, int32_t device, void* stream) {
    if (!X || !planes || !centroids_out || (mem != NOMAD_HOST && mem != NOMAD_DEVICE)) return NOMAD_E_INVALID_ARG;
    if (n < 1 || d < 1 || d > NOMAD_KNN_MAX_DIM || K < 1 || K > n || n_planes < 1 || n_planes > kMaxPlanes || device < 0) return NOMAD_E_INVALID_ARG;
    if (((int64_t)1 << n_planes) < K) return NOMAD_E_INVALID_ARG;
    if (n >= ((int64_t)1 << 31) - 256) return NOMAD_E_TOO_LARGE;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return NOMAD_E_HIP;
    KTRY(hipSetDevice(device));
    hipStream_t st = (hipStream_t)stream;
    Buffers buf(st);
    const float *dX = X, *dP = planes;
    const int32_t* dA = anchors;
    float* dC = centroids_out;
    int32_t* dB = buckets_out;
    std::vector<int32_t> hanchors((size_t)n_planes, 0);
    if (mem == NOMAD_HOST) {
        float *x = nullptr, *pl = nullptr, *c = nullptr;
        KTRY(buf.alloc(&x, (size_t)n * d));
        KTRY(buf.alloc(&pl, (size_t)n_planes * d));
        KTRY(buf.alloc(&c, (size_t)K * d));
        KTRY(hipMemcpyAsync(x, X, sizeof(float) * (size_t)n * d, hipMemcpyHostToDevice, st));
        KTRY(hipMemcpyAsync(pl, planes, sizeof(float) * (size_t)n_planes * d, hipMemcpyHostToDevice, st));
        dX = x; dP = pl; dC = c;
        if (anchors) {
            int32_t* a = nullptr;
            KTRY(buf.alloc(&a, (size_t)n_planes));
            KTRY(hipMemcpyAsync(a, anchors, sizeof(int32_t) * (size_t)n_planes, hipMemcpyHostToDevice, st));
            for (int32_t j = 0; j < n_planes; ++j) hanchors[j] = anchors[j];
            dA = a;
        }
    } else if (anchors) {
        KTRY(hipMemcpyAsync(hanchors.data(), anchors, sizeof(int32_t) * (size_t)n_planes, hipMemcpyDeviceToHost, st));
        KTRY(hipStreamSynchronize(st));
    }
    for (int32_t j = 0; j < n_planes; ++j)
        if (hanchors[j] < 0 || hanchors[j] >= n) return NOMAD_E_INVALID_ARG;   // an anchor that is no data point
    if (!anchors) {   // every plane through the median of a sample along its normal
        int32_t* a = nullptr;
        KTRY(buf.alloc(&a, (size_t)n_planes));
        double* proj = nullptr;
        KTRY(buf.alloc(&proj, (size_t)n_planes * kLshSample));
        hipLaunchKernelGGL(k_lsh_projections, dim3((uint32_t)n_planes, kLshSample / 64), dim3(64), 0, st, dX, n, d, dP, proj);
        hipLaunchKernelGGL(k_lsh_median_anchors, dim3((uint32_t)n_planes), dim3(kLshSample), 0, st, (const double*)proj, n, a);
        dA = a;
    }
    if (!dB || mem == NOMAD_HOST) {
        int32_t* bk = nullptr;
        KTRY(buf.alloc(&bk, (size_t)n));
        dB = bk;
    }
    MeanStep m_step;
    {
        int rc = m_step.init(buf, n, K, d);
        if (rc) return rc;
    }
    double* table = nullptr;   // normals, then offsets
    KTRY(buf.alloc(&table, (size_t)32 * d + 3 * 32));
    const auto buckets = [&](auto planes_of) {
        constexpr int P = decltype(planes_of)::value;
        double* offset = table + (size_t)P * d;
        hipLaunchKernelGGL(k_lsh_table<P>, dim3(P), dim3(256), 0, st, dX, d, dP, dA, n_planes, table, offset);
        const auto launch = [&](auto kernel, int shared) {
            hipLaunchKernelGGL(kernel, dim3(blocks_of(n, 256 / shared)), dim3(256), 0, st, dX, n, d, dP, dA, (const double*)table, (const double*)offset, n_planes, K, dB);
        };
        const int shared = lsh_shared(n, d, P);
        if (shared == 1) launch(k_lsh_buckets<P, 1>, shared);
        else if (shared == 2) launch(k_lsh_buckets<P, 2>, shared);
        else launch(k_lsh_buckets<P, 4>, shared);
    };
    if (n_planes <= 8) buckets(std::integral_constant<int, 8>());
    else if (n_planes <= 16) buckets(std::integral_constant<int, 16>());
    else buckets(std::integral_constant<int, 32>());
    hipLaunchKernelGGL(k_lsh_fallback, dim3(blocks_of((int64_t)K * d, 256)), dim3(256), 0, st, dX, n, d, K, dC);
    // bucket means: the M step of Lloyd's iteration on the buckets
    {
        uint32_t* n_list = nullptr;
        KTRY(buf.alloc(&n_list, 1));
        KTRY(hipMemsetAsync(n_list, 0, sizeof(uint32_t), st));
        int rc = m_step.small ? NOMAD_OK : m_step.sort(st, (const int32_t*)dB);
        if (rc) return rc;
        rc = m_step.small ? m_step.small_means(st, dX, (const int32_t*)dB, nullptr, dC, nullptr, nullptr) : m_step.means(st, dX, dC, n_list);
        if (rc) return rc;
    }
    KTRY(hipGetLastError());
    if (mem == NOMAD_HOST) {
        KTRY(hipMemcpyAsync(centroids_out, dC, sizeof(float) * (size_t)K * d, hipMemcpyDeviceToHost, st));
        if (buckets_out) KTRY(hipMemcpyAsync(buckets_out, dB, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, st));
    }
    KTRY(hipStreamSynchronize(st));
    return NOMAD_OK;
}

namespace {

// Exact k nearest other points, among all n rows of A, of the rows listed in dQ (m of them; nullptr: every row).
// out [m * k] on the device.  A workgroup of the filter scans every candidate of its group, so few queries would leave
// most of the chip idle: the candidates are then cut into slices, every slice is a group of its own with a copy of the
// queries, and the per-slice answers are merged by exact distance.
int neighbours_of_queries(hipStream_t st, Buffers& buf, const float* A, int64_t n, int32_t d, const int32_t* dQ, int64_t m, int32_t k,
                          int32_t* out) {
    const int32_t list_len = k + kPad;
    const int64_t block_queries = 8 * knn_tile(d, list_len);
    const int64_t base_blocks = (m + block_queries - 1) / block_queries;
    // as many slices as fill the compute units' last round best: rounds of 256 workgroups times a slice's length
    const int64_t most = std::min<int64_t>(256 / k, std::max<int64_t>(1, n / 4096));   // the merge ranks slices * k candidates in one
    int64_t G = 1;                                                                       // workgroup; slices of at least 4,096 candidates
    const auto rounds_cost = [&](int64_t g) { return (double)((base_blocks * g + 255) / 256) * (double)((n + g - 1) / g); };
    for (int64_t g = 2; g <= most; ++g)
        if (rounds_cost(g) < 0.98 * rounds_cost(G)) G = g;
    const int64_t slice = (n + G - 1) / G, mq = m * G;
    if (mq >= ((int64_t)1 << 31) - 256) return NOMAD_E_TOO_LARGE;
    uint32_t *max_q = nullptr, *max_c = nullptr, *n_flagged = nullptr;
    int32_t *cand = nullptr, *flagged = nullptr, *self = nullptr, *group_of_q = nullptr, *slice_of = nullptr, *part = nullptr;
    float *cnorm = nullptr, *qnorm = nullptr, *keys = nullptr, *tau = nullptr, *centre = nullptr, *AQ = nullptr;
    int* bad = nullptr;
    uint8_t* zeroed = nullptr;   // max_q, max_c, bad, n_flagged, centre
    const size_t zero_words = ((size_t)2 * G + 2 + 3) / 4 * 4;   // ahead of the centres, whose rows are read 16 bytes at a time
    const size_t zero_bytes = sizeof(uint32_t) * (zero_words + (size_t)G * d);
    KTRY(buf.alloc(&zeroed, zero_bytes));
    KTRY(hipMemsetAsync(zeroed, 0, zero_bytes, st));
    max_q = (uint32_t*)zeroed; max_c = max_q + G; bad = (int*)(max_c + G); n_flagged = (uint32_t*)(bad + 1); centre = (float*)zeroed + zero_words;
    KTRY(buf.alloc(&cand, (size_t)mq * list_len)); KTRY(buf.alloc(&keys, (size_t)mq * list_len)); KTRY(buf.alloc(&flagged, (size_t)mq)); KTRY(buf.alloc(&tau, (size_t)mq));
    KTRY(buf.alloc(&cnorm, (size_t)n)); KTRY(buf.alloc(&AQ, (size_t)mq * d));
    KTRY(buf.alloc(&self, (size_t)mq));
    std::vector<uint32_t> hq((size_t)G + 1), hc((size_t)G + 1);
    const int32_t slab_rows = centroid_rows(n);
    std::vector<KnnBlock> hslabs;
    for (int64_t g = 0; g <= G; ++g) {
        hq[g] = (uint32_t)(g * m);
        hc[g] = (uint32_t)std::min<int64_t>(n, g * slice);
    }
    for (int64_t g = 0; g < G; ++g)
        for (int64_t q0 = 0; q0 < (int64_t)(hc[g + 1] - hc[g]); q0 += slab_rows) hslabs.push_back(KnnBlock{(int32_t)g, (int32_t)q0});
    PackedSide qside, cside;
    qside.plan(hq, d, list_len);
    cside.plan(hc, d, list_len);
    const int waves = knn_filter_waves(qside.tile, qside.n_tiles);
    const std::vector<KnnBlock> hblocks = filter_blocks(qside, cside, waves);
    HostArrays up;
    const size_t at_q = up.add(hq), at_c = up.add(hc), at_qt = up.add(qside.tstart), at_ct = up.add(cside.tstart), at_blocks = up.add(hblocks),
                 at_slabs = up.add(hslabs);
    KTRY(up.upload(buf, st));
    const uint32_t *qstart = up.at<uint32_t>(at_q), *cstart = up.at<uint32_t>(at_c);
    const KnnBlock *blocks = up.at<KnnBlock>(at_blocks), *slabs = up.at<KnnBlock>(at_slabs);
    qside.d_start = qstart; qside.d_tstart = up.at<uint32_t>(at_qt);
    cside.d_start = cstart; cside.d_tstart = up.at<uint32_t>(at_ct);
    if (int rc = qside.alloc(buf, false)) return rc;
    if (int rc = cside.alloc(buf, true)) return rc;
    const int64_t lists = G * (64 / qside.tile);   // lanes that hold candidates of one query
    const int32_t share_rank = (int32_t)((list_len + 2 * lists - 1) / (2 * lists));
    const int lanes_list = knn_list_class(qside.tile, list_len);
    const bool share = slices_share(G, slice, qside.tile, list_len > kShortList) && knn_shares(qside.tile, qside.steps, lanes_list) && 4 * share_rank <= lanes_list;
    float4* shared = nullptr;
    if (share) {
        KTRY(buf.alloc(&qnorm, (size_t)mq));
        const size_t words = (size_t)mq * (64 / qside.tile);
        KTRY(buf.alloc(&shared, words));
        KTRY(hipMemsetAsync(shared, 0x7f, sizeof(float4) * words, st));   // 3.4e38: bounds nothing
    }
    if (G > 1) {
        KTRY(buf.alloc(&group_of_q, (size_t)mq));
        KTRY(buf.alloc(&slice_of, (size_t)n));
        KTRY(buf.alloc(&part, (size_t)mq * k));
        hipLaunchKernelGGL(k_periodic_ids, dim3(blocks_of(n, 256)), dim3(256), 0, st, (const int32_t*)nullptr, slice, n, slice_of, (int32_t*)nullptr);
    }
    // every slice centred on its own mean; the largest centred norm of a group covers its candidates and its queries
    hipLaunchKernelGGL(k_periodic_ids, dim3(blocks_of(mq, 256)), dim3(256), 0, st, dQ, m, mq, group_of_q, self);
    hipLaunchKernelGGL(k_gather_rows, dim3(blocks_of(mq * d, 256)), dim3(256), 0, st, A, n, d, dQ, m, mq, AQ, bad);
    int hbad = 0;
    KTRY(hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, st));
    KTRY(hipStreamSynchronize(st));
    if (hbad) return NOMAD_E_INVALID_ARG;   // a query outside 0..n-1
    hipLaunchKernelGGL(k_knn_centroid_sums, dim3((uint32_t)hslabs.size()), dim3(256), 0, st, A, d, (const int32_t*)nullptr, cstart, slabs, slab_rows, centre);
    hipLaunchKernelGGL(k_knn_centroid_finish, dim3(blocks_of(G * d, 256)), dim3(256), 0, st, centre, cstart, (int32_t)G, d);
    launch_norms(st, A, n, d, nullptr, slice_of, centre, cnorm, max_c);
    launch_norms(st, AQ, mq, d, nullptr, group_of_q, centre, qnorm, max_q);
    cside.fill(st, A, d, nullptr, centre, max_c, max_q, cnorm);
    qside.fill(st, AQ, d, nullptr, centre, max_q, nullptr, nullptr);
    KnnSets P{};
    P.XQ = AQ; P.XC = A; P.qmembers = nullptr; P.cmembers = nullptr; P.qstart = qstart; P.cstart = cstart;
    P.Q = qside.view(max_q); P.C = cside.view(max_c); P.centre = centre; P.group_of_q = group_of_q; P.n_q = mq; P.n_c = n; P.d = d; P.same_set = 0; P.chunk = knn_chunk_columns(d, list_len);
    P.self_row = self;
    if (share) {
        P.shared = shared; P.q_norm = qnorm; P.slices = (int32_t)G; P.share_rank = share_rank;
    }
    int rc = nearest_in_groups(st, buf, P, blocks, (uint32_t)hblocks.size(), waves, k, cand, keys, tau, flagged, n_flagged, G > 1 ? part : out);
    if (rc) return rc;
    if (G > 1) {
        hipLaunchKernelGGL(k_merge_slices, dim3((uint32_t)m), dim3(256), 0, st, (const float*)AQ, A, d, (const int32_t*)part, (int32_t)G, m, k, out);
        KTRY(hipGetLastError());
    }
    return NOMAD_OK;
}

// The same for rows of two columns and a few thousand points or more: a grid of cells (metrics_kernels.h).
constexpr int64_t kPlanePoints = 1024;
int neighbours_in_plane(hipStream_t st, Buffers& buf, const float* A, int64_t n, const int32_t* dQ, int64_t m, int32_t k, int32_t* out,
                        unsigned long long* bad) {
    const int32_t G = (int32_t)std::max<int64_t>(1, std::min<int64_t>(kMaxGrid, (int64_t)std::sqrt((double)n / kCellPoints)));
    const uint64_t cells = (uint64_t)G * G;
    const uint32_t n_tiles = (uint32_t)((cells + kScanTile - 1) / kScanTile);
    uint32_t *box = nullptr, *counts = nullptr, *tile_total = nullptr, *rank = nullptr;
    float2* pos = nullptr;
    int32_t* id = nullptr;
    KTRY(buf.alloc(&box, 4)); KTRY(buf.alloc(&counts, (size_t)cells)); KTRY(buf.alloc(&tile_total, (size_t)n_tiles));
    KTRY(buf.alloc(&rank, (size_t)n)); KTRY(buf.alloc(&pos, (size_t)n)); KTRY(buf.alloc(&id, (size_t)n));
    KTRY(hipMemsetAsync(counts, 0, sizeof(uint32_t) * (size_t)cells, st));
    hipLaunchKernelGGL(k_plane_box_clear, dim3(1), dim3(64), 0, st, box);
    hipLaunchKernelGGL(k_plane_box, dim3((uint32_t)std::min<int64_t>(512, blocks_of(n, 256))), dim3(256), 0, st, A, n, box);
    hipLaunchKernelGGL(k_plane_count, dim3(blocks_of(n, 256)), dim3(256), 0, st, A, n, (const uint32_t*)box, G, counts, rank);
    hipLaunchKernelGGL(k_sort_scan_tiles, dim3(n_tiles), dim3(256), 0, st, counts, cells, tile_total);
    hipLaunchKernelGGL(k_sort_scan, dim3(1), dim3(1024), 0, st, tile_total, (uint64_t)n_tiles);
    hipLaunchKernelGGL(k_plane_place, dim3(blocks_of(n, 256)), dim3(256), 0, st, A, n, (const uint32_t*)box, G, (const uint32_t*)counts,
                       (const uint32_t*)tile_total, (const uint32_t*)rank, pos, id);
    hipLaunchKernelGGL(k_plane_neighbours, dim3(blocks_of(m, 4)), dim3(256), 0, st, A, n, dQ, m, k, (const uint32_t*)box, G, (const uint32_t*)counts,
                       (const uint32_t*)tile_total, (const float2*)pos, (const int32_t*)id, out, bad);
    KTRY(hipGetLastError());
    return NOMAD_OK;
}

}  // namespace

extern "C" int nomad_neighbourhood_preservation(const float* X, int64_t n, int32_t d, const float* Y, int32_t d_low, int32_t k,
                                                const int32_t* queries, int64_t n_queries, int64_t* hits_out, int mem, int32_t device,
                                                void* stream) {
    if (!X || !Y || !hits_out || (mem != NOMAD_HOST && mem != NOMAD_DEVICE)) return NOMAD_E_INVALID_ARG;
    if (n < 2 || d < 1 || d > NOMAD_KNN_MAX_DIM || d_low < 1 || d_low > NOMAD_KNN_MAX_DIM || k < 1 || k > NOMAD_KNN_MAX_K || device < 0)
        return NOMAD_E_INVALID_ARG;
    if (queries ? n_queries < 1 : (n_queries != 0 && n_queries != n)) return NOMAD_E_INVALID_ARG;
    if (n >= ((int64_t)1 << 31) - 256 || n_queries >= ((int64_t)1 << 31) - 256) return NOMAD_E_TOO_LARGE;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return NOMAD_E_HIP;
    KTRY(hipSetDevice(device));
    hipStream_t st = (hipStream_t)stream;
    const int64_t m = queries ? n_queries : n;
    const float *dX = X, *dY = Y;
    const int32_t* dQ = queries;
    Buffers io(st);
    if (mem == NOMAD_HOST) {
        float *x = nullptr, *y = nullptr;
        KTRY(io.alloc(&x, (size_t)n * d));
        KTRY(io.alloc(&y, (size_t)n * d_low));
        KTRY(hipMemcpyAsync(x, X, sizeof(float) * (size_t)n * d, hipMemcpyHostToDevice, st));
        KTRY(hipMemcpyAsync(y, Y, sizeof(float) * (size_t)n * d_low, hipMemcpyHostToDevice, st));
        dX = x; dY = y;
        if (queries) {
            int32_t* q = nullptr;
            KTRY(io.alloc(&q, (size_t)m));
            KTRY(hipMemcpyAsync(q, queries, sizeof(int32_t) * (size_t)m, hipMemcpyHostToDevice, st));
            dQ = q;
        }
    }
    int32_t *high = nullptr, *low = nullptr;
    unsigned long long* hits = nullptr;
    KTRY(io.alloc(&high, (size_t)m * k));
    KTRY(io.alloc(&low, (size_t)m * k));
    KTRY(io.alloc(&hits, 2));   // the count, and whether a query lies outside 0..n-1
    KTRY(hipMemsetAsync(hits, 0, 2 * sizeof(unsigned long long), st));
    const auto neighbours = [&](const float* A, int32_t dim, int32_t* to) {
        Buffers work(st);   // given back before the second space takes its own
        return dim == 2 && n >= kPlanePoints ? neighbours_in_plane(st, work, A, n, dQ, m, k, to, hits + 1) : neighbours_of_queries(st, work, A, n, dim, dQ, m, k, to);
    };
    if (int rc = neighbours(dX, d, high)) return rc;
    if (int rc = neighbours(dY, d_low, low)) return rc;
    unsigned long long hhits[2] = {0, 0};
    hipLaunchKernelGGL(k_overlap, dim3(blocks_of(m, 256)), dim3(256), 0, st, (const int32_t*)high, (const int32_t*)low, k, m, hits);
    KTRY(hipMemcpyAsync(hhits, hits, sizeof(hhits), hipMemcpyDeviceToHost, st));
    KTRY(hipGetLastError());
    KTRY(hipStreamSynchronize(st));
    if (hhits[1]) return NOMAD_E_INVALID_ARG;
    *hits_out = (int64_t)hhits[0];
    return NOMAD_OK;
}

namespace {

// One launch covers at most kTripletsPerLaunch triplets (262,144 workgroups), so that any count up to the documented
// 2^40 stays inside the grid limits; the launches add into the same counter.
constexpr int64_t kTripletsPerLaunch = (int64_t)1 << 24;

int check_triplet_arguments(const float* X, int64_t n, int32_t d, const float* Y, int32_t d_low, int64_t n_triplets,
                            const int64_t* agree_out, int32_t device) {
    if (!X || !Y || !agree_out) return NOMAD_E_INVALID_ARG;
    if (n < 3 || d < 1 || d_low < 1 || n_triplets < 0 || device < 0) return NOMAD_E_INVALID_ARG;
    if (n >= ((int64_t)1 << 31) - 256 || n_triplets > ((int64_t)1 << 40)) return NOMAD_E_TOO_LARGE;
    return NOMAD_OK;
}

// enqueue the count of the triplets 0 .. n_triplets-1 into *agree (device memory, cleared first by a kernel)
int enqueue_triplets(hipStream_t st, const float* dX, int32_t d, const float* dY, int32_t d_low, int64_t n, int64_t n_triplets,
                     uint64_t seed, unsigned long long* agree) {
    hipLaunchKernelGGL(k_store_u64, dim3(1), dim3(64), 0, st, agree, 0ull);
    const auto kernel = d >= kStagedColumns ? k_triplets<true> : k_triplets<false>;
    for (int64_t t0 = 0; t0 < n_triplets; t0 += kTripletsPerLaunch) {
        const int64_t t1 = std::min(n_triplets, t0 + kTripletsPerLaunch);
        hipLaunchKernelGGL(kernel, dim3(blocks_of(t1 - t0, 64)), dim3(64), 0, st, dX, d, dY, d_low, (uint32_t)n, t0, t1,
                           (uint32_t)seed, (uint32_t)(seed >> 32), agree);
    }
    KTRY(hipGetLastError());
    return NOMAD_OK;
}

// ---- work space of nomad_random_triplet_accuracy_noalloc: lives in the code object, one copy per device
constexpr int kScratchWords = 32;   // 256 bytes; word 0 is the agreement counter
static __device__ __align__(256) unsigned long long scratch[kScratchWords];

constexpr int kMaxScratchDevices = 64;
unsigned long long* scratch_address[kMaxScratchDevices];   // device address of `scratch` on every device, once asked for
std::mutex scratch_mutex;

// Device address of this device's copy of `scratch` (the device must be current).  The array's name is only a
// host-side handle: kernels and copies take the address hipGetSymbolAddress returns.
int scratch_on_device(int32_t device, unsigned long long** out) {
    if (device >= kMaxScratchDevices) return NOMAD_E_INVALID_ARG;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_address[device]) {
        void* p = nullptr;
        KTRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return NOMAD_E_HIP;
        scratch_address[device] = (unsigned long long*)p;
    }
    *out = scratch_address[device];
    return NOMAD_OK;
}

}  // namespace

extern "C" int nomad_random_triplet_accuracy(const float* X, int64_t n, int32_t d, const float* Y, int32_t d_low, int64_t n_triplets,
                                             uint64_t seed, int64_t* agree_out, int mem, int32_t device, void* stream) {
    if (mem != NOMAD_HOST && mem != NOMAD_DEVICE) return NOMAD_E_INVALID_ARG;
    if (int rc = check_triplet_arguments(X, n, d, Y, d_low, n_triplets, agree_out, device)) return rc;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return NOMAD_E_HIP;
    KTRY(hipSetDevice(device));
    hipStream_t st = (hipStream_t)stream;
    const float *dX = X, *dY = Y;
    Buffers buf(st);
    if (mem == NOMAD_HOST) {
        float *x = nullptr, *y = nullptr;
        KTRY(buf.alloc(&x, (size_t)n * d));
        KTRY(buf.alloc(&y, (size_t)n * d_low));
        KTRY(hipMemcpyAsync(x, X, sizeof(float) * (size_t)n * d, hipMemcpyHostToDevice, st));
        KTRY(hipMemcpyAsync(y, Y, sizeof(float) * (size_t)n * d_low, hipMemcpyHostToDevice, st));
        dX = x; dY = y;
    }
    unsigned long long* agree = nullptr;
    unsigned long long hagree = 0;
    KTRY(buf.alloc(&agree, 1));
    if (int rc = enqueue_triplets(st, dX, d, dY, d_low, n, n_triplets, seed, agree)) return rc;
    KTRY(hipMemcpyAsync(&hagree, agree, sizeof(hagree), hipMemcpyDeviceToHost, st));
    KTRY(hipStreamSynchronize(st));
    *agree_out = (int64_t)hagree;
    return NOMAD_OK;
}

extern "C" int nomad_random_triplet_accuracy_noalloc(const float* X, int64_t n, int32_t d, const float* Y, int32_t d_low,
                                                     int64_t n_triplets, uint64_t seed, int64_t* agree_out, int32_t device,
                                                     void* stream) {
    if (int rc = check_triplet_arguments(X, n, d, Y, d_low, n_triplets, agree_out, device)) return rc;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return NOMAD_E_HIP;
    KTRY(hipSetDevice(device));
    hipStream_t st = (hipStream_t)stream;
    unsigned long long* counter = nullptr;
    if (int rc = scratch_on_device(device, &counter)) return rc;
    unsigned long long hagree = 0;
    if (int rc = enqueue_triplets(st, X, d, Y, d_low, n, n_triplets, seed, counter)) return rc;
    KTRY(hipMemcpyAsync(&hagree, counter, sizeof(hagree), hipMemcpyDeviceToHost, st));
    KTRY(hipStreamSynchronize(st));
    *agree_out = (int64_t)hagree;
    return NOMAD_OK;
}
#pragma GCC visibility pop
