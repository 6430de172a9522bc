// libnomad: how the deterministic edge pass is laid out for a problem -- tile size, LDS budgets of the three edge-pass
// kernels, which of them runs, whether a round's records are sorted, the number of record phases.  Plain C++ with no
// device code and no HIP types, so that the rules can be compiled and checked on a machine without a GPU; the kernels'
// header includes it for the constants and LDS sizes they share with the host.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#if defined(__HIPCC__)
#define NOMAD_HOST_DEVICE __host__ __device__
#else
#define NOMAD_HOST_DEVICE
#endif

namespace nomad {

constexpr int kMaxTileBits = 13;        // 8192 points: 128 KB of accumulators in the tile pass
constexpr int kMinTileBits = 8;
constexpr int kMinFittedTileBits = 4;  // the smallest tile fit_tiles makes
constexpr int kChunk = 128;             // records per chunk (1.5 KB): every (workgroup, tile) chain ends in a partly filled
                                        // chunk, so the pool carries workgroups x tiles x kChunk records of slack
constexpr int kBinBlock = 1024;         // threads of the tile pass and of the large edge-pass workgroup
constexpr int kSmallBinBlock = 256;     // threads of the small one (fit_tiles)
constexpr int kMaxBinsPerThread = 8;    // tiles one thread owns in the per-round scan of the sorted form
constexpr size_t kMaxLdsBytes = 160 * 1024 - 256;   // per workgroup on gfx950, less the kernels' static LDS
constexpr int kDefaultFlushRounds = 2;  // unsorted binned edge pass: rounds between two flushes (5 % faster than one at
                                        // 60 M points; the records of four rounds do not fit the registers)

// ---- LDS of the edge-pass kernels
// binned: per tile (record count / first sorted slot, fill of the open chunk, open chunk, first chunk allocated this
// round) and, in the sorted form, the round's records sorted by tile
NOMAD_HOST_DEVICE inline size_t binned_records_per_round(int s, int block) { return (size_t)block * (s + 1) + 2 * (block / 64); }
NOMAD_HOST_DEVICE inline size_t binned_lds_bytes(uint32_t n_bins, int s, int block, bool sorted = true, int rounds = 1) {
    return ((size_t)4 * n_bins + 1 + (sorted ? 3 * rounds * binned_records_per_round(s, block) : 0)) * sizeof(uint32_t);
}
// pooled (16-bit picks): pool rows, points and 64-bit sums, the tile tables, the partial head sums of a block (two per
// wavefront and round)
NOMAD_HOST_DEVICE inline size_t pooled_side_records(int64_t block_edges) { return (size_t)(block_edges / 32); }
NOMAD_HOST_DEVICE inline size_t pooled_lds_bytes(uint32_t n_bins, int64_t block_edges, uint32_t pool_size) {
    return (size_t)pool_size * 28 + ((size_t)4 * n_bins + 3 * pooled_side_records(block_edges)) * sizeof(uint32_t);
}
// pooled with distinct picks: the same plus the starts of the next block's lines
NOMAD_HOST_DEVICE inline size_t distinct_lds_bytes(uint32_t n_bins, uint32_t pool_size, uint32_t lines, int rounds) {
    return (size_t)pool_size * 28 + ((size_t)lines + (size_t)4 * n_bins + 3 * (size_t)(32 * rounds)) * sizeof(uint32_t);
}

// exchanged edge pass (exchange_kernels.h): blocks of kExchangeLanes * R edges, whose references fit half of a compute unit's LDS.
// (All of it, one workgroup of 1,024 lanes that fetches the next block while it computes one: runs twice as long, but k_exchange_edges took
// 2.29 ms for 75 M edges where two workgroups take turns in 1.79, and 0.129 for 0.054 at 100 k points.)
constexpr int kExchangeLanes = 768;
constexpr uint32_t kExchangeSpare = 4096;        // slots that mean nothing, for lanes without a reference
constexpr uint32_t kExchangeTilesTogether = 16;  // neighbouring tiles that go to one XCD (32: the same; 64: 2.58 ms for 2.11, the XCDs' shares differ)
NOMAD_HOST_DEVICE constexpr uint32_t exchange_padded_tiles(uint32_t n) {
    return (n + 8 * kExchangeTilesTogether - 1) / (8 * kExchangeTilesTogether) * (8 * kExchangeTilesTogether);
}
NOMAD_HOST_DEVICE constexpr int exchange_edges_per_lane(int s) {
    const int r = (int)(78 * 1024 / (8 * (s + 1) * kExchangeLanes));
    return r < 1 ? 1 : r > 4 ? 4 : r;
}
NOMAD_HOST_DEVICE constexpr int exchange_block_edges(int s) { return kExchangeLanes * exchange_edges_per_lane(s); }
NOMAD_HOST_DEVICE constexpr size_t exchange_slots(int s) {   // one per reference, two per wavefront of head sums; a multiple of 64
    return ((size_t)exchange_block_edges(s) * (s + 1) + 2 * (exchange_block_edges(s) / 64) + 63) / 64 * 64;
}
NOMAD_HOST_DEVICE constexpr size_t exchange_deal_lds_bytes(int s, uint32_t n_tiles) { return exchange_slots(s) * 2 + (size_t)n_tiles * 4; }
NOMAD_HOST_DEVICE constexpr size_t exchange_edges_lds_bytes(int s) { return exchange_slots(s) * 8; }

// edge pass that leaves its forces in runs (run_kernels.h): blocks of runs_lanes * runs_edges_per_lane edges.  As many lanes in flight as registers allow with two
// workgroups and more a compute unit, an edge a lane; up to two negatives three edges a lane, for as long a run: 6 M points in groups, s = 2, edge pass and sums
// 2.78 + 1.60 ms with 1,024 x 1, 2.74 + 1.02 with 512 x 3, 3.87 + 1.06 with 512 x 4 and 4.73 + 1.02 with 512 x 5 (two workgroups of 61 and 77 KB), 3.24 + 1.40 with 768 x 2.
NOMAD_HOST_DEVICE constexpr int runs_lanes(int s) { return s > 2 && s <= 6 ? 1024 : 512; }
NOMAD_HOST_DEVICE constexpr int runs_edges_per_lane(int s) { return s <= 2 ? 3 : 1; }
NOMAD_HOST_DEVICE constexpr int runs_waves_per_simd(int s) { return runs_lanes(s) == 1024 ? 8 : s <= 2 ? 4 : 6; }
NOMAD_HOST_DEVICE constexpr int runs_block_edges(int s) { return runs_lanes(s) * runs_edges_per_lane(s); }
NOMAD_HOST_DEVICE constexpr size_t runs_slots(int s) {   // one per reference, two per wavefront of head sums; a multiple of 64
    return ((size_t)runs_block_edges(s) * (s + 1) + 2 * (runs_block_edges(s) / 64) + 63) / 64 * 64;
}
NOMAD_HOST_DEVICE constexpr size_t runs_lds_bytes(int s, uint32_t n_tiles) { return runs_slots(s) * 10 + (size_t)n_tiles * 4; }

// ---- the plan
struct EdgePlanRequest {
    int64_t n = 0, E = 0;
    int s = 0;
    // pooled sampler (pool_size 0: none); distinct: picks in different lines (modes 1 and 2)
    int32_t pool_size = 0, pool_block = 0, pool_line = 1;
    bool pool_distinct = false;
    bool grouped = false;       // some cells are approximated
    bool far = false;           // groups whose far cells are sampled
    int batches = 1;            // sub-steps of an epoch
    // nomad_tune (0 = the library's choice, except pool_kernel: 1 = use the pooled kernels)
    int tune_edge_block = 0, tune_wg_per_cu = 0, tune_pool_kernel = 1, tune_record_sort = 0, tune_flush_rounds = 0,
        tune_exchange = 0, tune_phases = 0;
};

struct EdgePlan {
    int tile_bits = kMinTileBits;
    uint32_t n_bins = 0;
    int bin_block = 0;          // lanes per workgroup of the edge pass; 0: its tables do not fit LDS
    int wg_per_cu = 1;
    bool sorted = true;         // a round's records are counting-sorted by tile in LDS before they are written
    int flush_rounds = 1;       // unsorted form: rounds between two flushes
    int pool_rounds = 0;        // > 0: a pooled edge pass runs, pool_block = 1024 * pool_rounds
    bool distinct_kernel = false;
};

inline EdgePlan plan_edge_pass(const EdgePlanRequest& q) {
    EdgePlan p;
    // about a thousand tiles when n allows, never above 8192 points a tile
    while (p.tile_bits < kMaxTileBits && (q.n >> p.tile_bits) > 1024) ++p.tile_bits;
    p.n_bins = (uint32_t)((q.n + ((int64_t)1 << p.tile_bits) - 1) >> p.tile_bits);
    // One persistent workgroup of 1024 lanes per compute unit: the more records a round sorts, the longer the
    // contiguous run each tile receives.  (Two workgroups of 512 per compute unit measured 17 % slower at
    // 10 M points; nomad_tune(NOMAD_TUNE_EDGE_BLOCK, 512) selects them for experiments when their LDS fits.)
    // A round's records are counting-sorted by tile in LDS before they are written, unless there are more tiles than
    // a round has records (60 M points, s = 2): then no tile receives a run worth sorting for, and every lane
    // writes its own records (two barriers and the scan over the tiles less per round).
    p.sorted = q.tune_record_sort != 2 && (q.tune_record_sort == 1 || (size_t)p.n_bins <= binned_records_per_round(q.s, 1024));
    if ((!p.sorted || p.n_bins <= (uint32_t)kMaxBinsPerThread * 1024) && binned_lds_bytes(p.n_bins, q.s, 1024, p.sorted) <= kMaxLdsBytes)
        p.bin_block = 1024;
    if (q.tune_edge_block == 512 && (!p.sorted || p.n_bins <= (uint32_t)kMaxBinsPerThread * 512) &&
        2 * (binned_lds_bytes(p.n_bins, q.s, 512, p.sorted) + 256) <= 160 * 1024) { p.bin_block = 512; p.wg_per_cu = 2; }
    if (q.tune_wg_per_cu) p.wg_per_cu = q.tune_wg_per_cu;
    // Pooled samplers: their own edge pass (pool in LDS) when the block is 1, 2, 4 or 8 rounds of 1024 positions, one
    // workgroup per compute unit.  (Two workgroups of 512 lanes per compute unit, which lets one block's
    // bookkeeping overlap the other's rounds, measured 4 % slower: the rounds are bound by vector-ALU issue.)
    if (q.pool_size > 0 && q.pool_block % 1024 == 0 && q.tune_pool_kernel) {
        const int r = q.pool_block / 1024;
        if (r == 1 || r == 2 || r == 4 || r == 8) {
            if (q.pool_distinct) {
                // 32-bit byte offsets into col / head (4 E) and theta (8 n)
                if (distinct_lds_bytes(p.n_bins, (uint32_t)q.pool_size, (uint32_t)(q.pool_size / q.pool_line), r) <= kMaxLdsBytes &&
                    q.E < ((int64_t)1 << 30) && q.n < ((int64_t)1 << 29)) { p.pool_rounds = r; p.distinct_kernel = true; }
            } else if (pooled_lds_bytes(p.n_bins, q.pool_block, (uint32_t)q.pool_size) <= kMaxLdsBytes) {
                p.pool_rounds = r;
            }
        }
    }
    if (p.pool_rounds) { p.bin_block = 1024; p.wg_per_cu = 1; p.sorted = true; }
    p.flush_rounds = (!p.sorted && p.bin_block == 1024) ? (q.tune_flush_rounds ? q.tune_flush_rounds : kDefaultFlushRounds) : 1;
    return p;
}

// plan_edge_pass makes up to a thousand tiles of at least 256 points.  What serves the tile pass is one tile per compute unit:
//   fewer points a tile in small problems (2,000 points in 8 tiles left 248 units idle: tile pass 32 us a step; 125 tiles of 16: 10.5 us);
//   in the sorted form more points a tile in large ones: the records a round brings to a tile are one contiguous run in memory,
//   and runs of 25 records instead of six end in fewer partial lines (1 M points, s = 5, a thousand tiles -> 245: edge pass
//   1.26 -> 1.12 ms, tile pass 0.32 -> 0.24; 123 tiles: tile pass 0.31).
// special_kernel: the edge pass is one of the kernels that know their options.  Those also come
//   with two rounds to a flush, where the records fit LDS (where chains are asked for, or runs do not fit; half the barriers and table passes: 100 k points 0.149 -> 0.142 ms,
//   6 M points in groups, s = 2, 4.26 -> 4.06);
//   with 256 lanes, for graphs of no more positions than give every compute unit one such workgroup (embeddings of
//   up to 10,224 points take plan_small's pass, and plan_runs leaves the sparsest graphs of the others to chains: those are what comes here, and what asks for chains):
//   one round is all there is, and its length goes with the lanes that share its barriers and LDS (whole epoch, 14 k edges: 22.0 -> 12.7 us, 58 k: 22.4 -> 18.8; with two such workgroups per compute unit 87 k: 24.0 -> 25.8, 116 k: 25.7 -> 29.9).
inline bool edge_tables_fit(const EdgePlan& p, const EdgePlanRequest& q) {
    const size_t lds = p.distinct_kernel ? distinct_lds_bytes(p.n_bins, (uint32_t)q.pool_size, (uint32_t)(q.pool_size / q.pool_line), p.pool_rounds)
                       : p.pool_rounds  ? pooled_lds_bytes(p.n_bins, q.pool_block, (uint32_t)q.pool_size)
                                        : p.wg_per_cu * binned_lds_bytes(p.n_bins, q.s, p.bin_block, p.sorted, p.flush_rounds);
    return lds <= kMaxLdsBytes;
}
inline void fit_tiles(EdgePlan& p, const EdgePlanRequest& q, int compute_units, bool special_kernel = true) {
    if (!p.bin_block) return;
    const auto tiles = [&](int bits) { return (uint32_t)((q.n + ((int64_t)1 << bits) - 1) >> bits); };
    if (p.sorted && !p.pool_rounds)
        while (p.tile_bits < kMaxTileBits && (q.n >> p.tile_bits) > compute_units) ++p.tile_bits;
    p.n_bins = tiles(p.tile_bits);
    while (p.tile_bits > kMinFittedTileBits && tiles(p.tile_bits - 1) <= (uint32_t)compute_units) {
        EdgePlan finer = p;
        finer.n_bins = tiles(--finer.tile_bits);
        if (!edge_tables_fit(finer, q)) break;
        p = finer;
    }
    if (!p.sorted || p.pool_rounds || !special_kernel) return;
    if (q.tune_edge_block == 0 && q.tune_wg_per_cu == 0 && q.E <= (int64_t)compute_units * kSmallBinBlock) {
        p.bin_block = kSmallBinBlock;
        p.wg_per_cu = 1;
    }
    if (p.bin_block == 1024 && binned_lds_bytes(p.n_bins, q.s, 1024, true, 2) <= kMaxLdsBytes)
        p.flush_rounds = 2;
}

// Record phases: the edge pass of a step runs over `phases` ranges of positions, each followed by the tile pass, so the
// pool holds the records of one range.  Default: as many (a power of two, at most 64) as keep one range's records under
// 8 GB, and under 4 GB for a step with more than 32 GB of records, where the pool would otherwise outweigh the graph
// (each further phase costs about half a per cent of an epoch: the tile pass walks shorter chains and carries its sums
// through memory).  Never more phases than the positions have blocks.
inline int plan_record_phases(int64_t E, int s, int bin_block, int tune_phases) {
    int phases = tune_phases;
    if (phases == 0) {
        const double step_bytes = (double)E * (s + 1) * 12.0;
        const double per_phase = step_bytes > 32e9 ? 4e9 : 8e9;
        phases = 1;
        while (phases < 64 && step_bytes / phases > per_phase) phases *= 2;
    }
    const int64_t blocks = (E + bin_block - 1) / bin_block;
    if (phases > blocks) phases = (int)blocks;
    return phases < 1 ? 1 : phases;
}

// Whether a problem takes the edge pass that sums in LDS (small_kernels.h), and its workgroups (0: no).  Embeddings whose sums fit
// one workgroup's LDS: whole epoch, records -> sums in LDS, us: 2,000 points and 47 k positions 19.1 -> 10.4 (s = 2: 17.0 -> 9.8, s = 8: 21.6 -> 11.8),
// 5,000 29.7 -> 17.4, 8,000 33.2 -> 21.5, 10,000 39.6 -> 26.0 (80 k positions, s = 2: 22.5 -> 18.1).
// Workgroups: a round of 1,024 positions costs 3.8 us, a megabyte of sums written and read back half of one: as many workgroups as there are
// rounds until their sums are 12 MB (8,000 points: 6 MB 25.8 us, 12 MB 21.5, 16 MB 21.9; 5,000: 16.8, 17.4, 17.6).  Where that makes some
// do two rounds, half as many as there are rounds do two each, with half the sums (0.85 to 0.96 of an epoch of 5,000 to 10,200 points).
// Not where so few workgroups (fewer than 150: from 5,243 points on) have more to do than what records cost on all compute units:
//   sampled far field, whose rounds are long (negatives are resolved one by one).  Rounds of a workgroup here / with records, time over that
//   of records, s = 2: 8,000 points 3 / 1 0.84, 10 / 4 0.99, 20 / 8 1.06, 10,200 8 / 3 0.96, 6 / 2 1.04, 26 / 9 1.26, 33 / 10 1.44; s = 5: 6,000 6 / 3
//   0.89, 8,000 4 / 2 0.96, 5 / 2 1.04, 20 / 8 1.25; s = 8: 6,000 3 / 2 0.86, 8,000 4 / 2 0.98, 5 / 2 1.11, 20 / 8 1.32; with fewer than 96 workgroups
//   (from 8,192 points) s = 5 and 8 2 / 1 1.01 to 1.24, 4 / 2 0.97 to 1.03;
//   no negatives, where records are one an edge: one round a workgroup, sums of up to 8 MB 0.71 to 0.92, 9 to 14 MB 1.04 to 1.13; two
//   rounds 0.75 to 0.92, with fewer than 96 workgroups 1.00 to 1.19; more 0.85 to 1.0.
// (All others: 0.45 to 0.99; s = 1 at 10,200 points up to 1.05.)
constexpr int kSmallLanes = 1024;
NOMAD_HOST_DEVICE inline size_t small_lds_bytes(int64_t n) { return (size_t)n * 16; }
inline int plan_small(const EdgePlanRequest& q, const EdgePlan& p, int compute_units) {
    const bool sorted_asked = q.tune_edge_block || q.tune_wg_per_cu || q.tune_record_sort || q.tune_flush_rounds || q.tune_phases || q.tune_exchange;
    if (q.s < 0 || q.s > 8 || q.E < 1 || q.pool_size || !p.bin_block || sorted_asked || q.n < 1 || small_lds_bytes(q.n) > kMaxLdsBytes) return 0;
    const int64_t rounds = (q.E + kSmallLanes - 1) / kSmallLanes, room = (int64_t)(12 << 20) / (int64_t)small_lds_bytes(q.n);
    const int64_t per = (rounds + room - 1) / room, records_per = (rounds + compute_units - 1) / compute_units;   // rounds of a workgroup
    if (room < 150) {
        if (q.far && q.s <= 3 && records_per > 4 && 2 * per >= 5 * records_per) return 0;
        if (q.far && q.s > 3 && (per > 2 * records_per || (room < 96 && per == 2))) return 0;
        if (q.s == 0 && rounds * (int64_t)small_lds_bytes(q.n) > (8 << 20) && (per == 1 || (room < 96 && per == 2))) return 0;
    }
    int64_t wg = rounds < room ? rounds : room;
    if (per == 2 && room < compute_units) wg = (rounds + 1) / 2;
    return (int)(wg < compute_units ? wg : compute_units);
}

// Whether a problem of one population takes the exchanged edge pass (exchange_kernels.h), and its tile kernels' shapes.
//   Which: embeddings beyond two L2s.  The sorted pass gathers a row per negative, and once most gathers miss the L2s they end
//   at 58 G lines/s; the exchange moves 42 bytes a reference in streams instead.  Time of an epoch, exchange over sorted, of the slowest
//   order of points (numbered cluster by cluster, 15 out-neighbours, symmetrised or not) and of a random one: s = 3, 5, 6, 8 at 800 k points
//   0.98, 0.97, 1.11, 1.02 (random 0.86 to 0.99), 900 k 0.95, 0.91, 0.99, 0.96 (0.79 to 0.90), 1 M 0.90, 0.87, 0.93, 0.91 (0.76 to 0.84), 1.06 M
//   0.97, 0.94, 0.97, 0.90 (0.84 to 0.88), 1.2 M 0.93, 0.91, 0.99, 0.91, 2 M 0.79, 0.73, -, 0.74.  s = 2 (fewer gathers an edge, the same
//   streams of heads and tails) 1 M 0.95 (0.76), 1.2 M 1.01 (0.91), 1.4 M 0.93 (0.80), 1.5 M 0.91 (0.76), 2 M 0.82; s = 1 1.2 M 1.09 (0.84), 1.5 M
//   1.04 (0.77), 1.8 M 1.01 (0.71), 2 M 0.95.  Smaller ones lose, s = 5 and 8: 100 k 1.07 and
//   1.13, 300 k 1.16 and 1.21, 600 k 1.08 and 1.12.  Up to where a run is shorter than two
//   references: s = 2 at 40 M points 28.9 -> 28.4 ms, s = 5 62.5 -> 55.5.
//   Sub-steps: where points are numbered cluster by cluster the tails of a sub-step lie in a stretch of the tiles, one workgroup of
//   k_tile_sums each, and few blocks leave compute units idle.  Exchange over sorted by millions of references a sub-step,
//   s = 2: 1 M points 1.4 / 1.08 / 1.03 at 2 / 5.6 / 6.4, 2 M 1.18 / 1.01 / 0.83 at 3.2 / 6.4 / 11; s = 3: 1 M 1.25 / 1.05 / 0.9 at 3.2 / 6.3 / 9.2;
//   s = 5: 1 M 1.24 / 1.07 / 0.81 at 1.9 / 4.6 / 11, 5 M 0.86 / 0.73 at 7.5 / 22; s = 8: 5 M 1.28 / 1.04 / 0.83 at 6.9 / 8.4 / 17; s = 1: 2 M 1.27 / 1.04 / 0.90 at
//   5 / 10 / 15.  (Random order: 2 M, s = 2 0.91 at 3.8, 1.42 at 1.4.)  The line is at 8.
//   Rows: runs of about seven references (10 M points) leave as partial sectors; two neighbouring tiles in LDS make them twice
//   as long (2.79 -> 2.45 ms for 75 M edges; at 5 M points a tile alone is as fast).
//   Lanes: as many as most runs have references (75 M edges, rows, 16 / 32 / 64 lanes: runs of 7.5 in pairs 2.67 / 2.47 / 2.76 ms, of 15
//   4.02 / 2.13 / 2.28, of 25 - / 1.99 / 1.95).  Sums, lanes of two references: runs of 7.5 4 / 8 / 16 lanes 2.32 / 2.14 / 2.18 ms; of 37 8 / 16
//   lanes 0.327 / 0.268 (a run is one segment or two).
struct ExchangePlan {
    bool use = false;
    bool pairs = false;                     // k_exchange_rows holds two neighbouring tiles
    int rows_lanes = 64;                    // lanes that take one run
    int sums_lanes = 16;                    // lanes that take a segment of twice as many references
    uint32_t parts = 1;                     // workgroups per tile (or pair) that answer
    int tile_bits = 0;
};
inline size_t exchange_rows_lds_bytes(const ExchangePlan& x) { return (size_t)8 << (x.tile_bits + (x.pairs ? 1 : 0)); }
// k_tile_sums: segments that a wavefront can have queued (8 bytes each), two steps of 64 / lanes and a round of 64; the tile's sums and all queues
constexpr uint32_t tile_sums_queue(int lanes) { return 2u * (64u / (uint32_t)lanes) + 64u; }
inline size_t tile_sums_lds_bytes(const ExchangePlan& x) { return ((size_t)16 << x.tile_bits) + (size_t)(kBinBlock / 64) * tile_sums_queue(x.sums_lanes) * 8; }
constexpr double kExchangeStepReferences = 8e6;
inline ExchangePlan plan_exchange(const EdgePlanRequest& q, const EdgePlan& p) {
    ExchangePlan x;
    if (q.s < 1 || q.s > 8 || q.E < 1 || q.pool_size || !p.bin_block || q.tune_exchange == 2) return x;
    const double run = (double)exchange_block_edges(q.s) * (q.s + 1) / p.n_bins;   // mean length of a run
    const bool sorted_asked = q.tune_edge_block || q.tune_wg_per_cu || q.tune_record_sort || q.tune_flush_rounds;
    const bool long_steps = q.batches <= 1 || (double)q.E * (q.s + 1) >= kExchangeStepReferences * q.batches;
    x.use = q.tune_exchange == 1 || (!sorted_asked && q.n >= (q.s < 3 ? 1500000 : 1000000) && long_steps && run >= 2);
    if (exchange_deal_lds_bytes(q.s, p.n_bins) > kMaxLdsBytes) x.use = false;
    x.tile_bits = p.tile_bits;
    x.pairs = run < 12;
    x.rows_lanes = x.pairs ? (2 * run < 9 ? 16 : 32) : run < 26 ? 32 : 64;
    x.sums_lanes = run < 12 ? 8 : 16;
    const uint32_t units = x.pairs ? (p.n_bins + 1) / 2 : p.n_bins;
    x.parts = units >= 512 ? 2 : (1024 + units - 1) / units;   // (four workgroups per compute unit and more at a few hundred tiles)
    return x;
}

// Whether a problem takes the edge pass that leaves its forces in runs (run_kernels.h), and the lanes of a segment of k_tile_sums.
//   Which: all that would otherwise leave records in chains, sorted by tile.  Time of an epoch, runs over chains (symmetrised, 12 to 15 out-neighbours,
//   numbered cluster by cluster): s = 5 10 k points 0.71, 20 k 0.67, 100 k 0.65, 300 k 0.71, 600 k 0.78, 900 k 0.83; s = 8 0.76 (100 k), 0.86 (900 k); s = 3 0.70 (400 k in
//   sub-steps), 0.82 (900 k); s = 2 0.71 (100 k), 0.79, 1.4 M 0.90; s = 1 0.79, 0.78 (600 k); none 0.74 (20 k), 0.86 (5 M); 64 sub-steps of 20 k to 5 M 0.57 to 0.85; every cluster its own
//   group 150 k 0.57, 1 M 0.76, 3 M (s = 2) 0.83, 8 M 0.94.
//   Not for graphs of so few edges that they are a few blocks (runs_sparse): a workgroup of chains then has 256 positions, a block of runs up to 1,536, and both are one chain of
//   loads.  Runs over chains at 4 k, 16 k, 32 k, 48 k edges, s = 2: 20 k points 1.26, 1.20, 1.09, 0.85, 900 k 1.35, 1.24, 1.13, 0.99 (in groups 1.21, 1.19, 1.14, 1.05; sampled means 1.32, 1.31,
//   1.22, 1.08); s = 1: 20 k 1.14, 1.07, 1.00, 0.82, 2 M 1.24, 1.19, 1.12, 0.97; s = 5: 20 k 1.09, 1.02, 0.90, 200 k 1.24, 1.12, 1.03, 0.89, 900 k 1.21, 1.10, 1.07, 0.94; s = 3: 20 k 1.02, 0.97, 0.87,
//   200 k 1.14, 1.04, 0.97, 900 k 1.12, 1.04, 0.99; none: 20 k 0.99, 0.95, 200 k 1.09, 1.02, 0.95, 2 M 1.19, 1.12, 1.07, 0.93.  s = 7 and 8 (blocks of 512): 0.60 to 1.0, two million points up to 1.06.  (Smaller
//   embeddings take sums in LDS.)
//   The exchange from a million points on (plan_exchange): runs take 0.94 to 1.0 of its time there, 1.03 to 1.09 at 1.3 M and 1.2 to 1.4 at 2.5 M, and in
//   random order 1.08, 1.11 and 1.5, so its lines stay.
//   Not with sampled means beyond 256 tiles: what a block's slots are made for are negatives, few of which get a force there, and the tiles look for their runs in many
//   blocks.  400 k 0.78 to 0.85, 1 M 0.90, 2 M 0.97, 2.5 M (s = 8) 1.03, 3 M (s = 5) 1.01, 5 M (s = 2) 1.02.
//   Nor where two workgroups do not fit a compute unit's LDS (77 KB a workgroup: 1.5 times as long as 46 KB with the same lanes in flight).
//   Tiles: one workgroup of k_tile_sums each, so as many as fill the compute units, of any number of points of eight bits (powers of two are tried first: kept where the
//   last round is 84 % full).  Whole epochs, powers of two over that: 147 tiles of 256 (300 k points) 1.04, 159 1.04, 196 1.03, in 64 sub-steps 306 of 512 1.06, groups of 150 k 1.07,
//   367 of 512 1.06; 220 of 256 0.99, 733 of 768 0.99.  Twice as many tiles: 0.87 to 1.02 (runs half as long), but 1.15 in short sub-steps.
//   Lanes of a segment (two references each): half of the mean run, us at 100 k points, s = 5, runs of 31 / 24 / 16: 8 lanes 63, 60, 52, 16 lanes 45, 39, 41, 32 lanes 36, 41, 57.
//   With groups a block's references lie in the tiles of its own clusters, whatever the mean: 6 M points, s = 2, 8 / 16 / 32 lanes 1.41 / 1.09 / 1.02 ms.
struct RunsPlan {
    bool use = false;
    int sums_lanes = 32;
    uint32_t n_tiles = 0, points = 0;   // of a tile: factor << shift
    uint32_t factor = 0, magic = 0;     // points / factor = 2^shift; x / factor = the high word of x magic, where x factor < 2^32
    int shift = 0;
};
NOMAD_HOST_DEVICE inline uint32_t runs_tile_of(uint32_t pt, int shift, uint32_t magic) {
    const uint32_t x = pt >> shift;
    return magic ? (uint32_t)(((uint64_t)x * magic) >> 32) : x;
}
inline bool runs_sparse(const EdgePlanRequest& q, int compute_units) {
    const int64_t few = q.s == 1 || q.s == 2 || q.n >= (1 << 19) ? 128 : q.n >= (1 << 17) ? 64 : 32;   // positions a compute unit
    return q.s <= 6 && small_lds_bytes(q.n) > kMaxLdsBytes && q.E <= few * compute_units;
}
inline RunsPlan plan_runs(const EdgePlanRequest& q, const EdgePlan& p, int compute_units = 256) {
    RunsPlan x;
    const bool records_asked = q.tune_edge_block || q.tune_wg_per_cu || q.tune_record_sort || q.tune_flush_rounds;
    if (q.s < 0 || q.s > 8 || q.E < 1 || q.pool_size || !p.bin_block || records_asked) return x;
    const int64_t most = (int64_t)1 << kMaxTileBits, rounds = ((int64_t)p.n_bins + compute_units - 1) / compute_units;
    const auto tiles_of = [&](int64_t points, uint32_t factor, int shift) {
        x.points = (uint32_t)points; x.factor = factor; x.shift = shift;
        x.magic = factor > 1 ? (uint32_t)(((uint64_t)1 << 32) / factor) + 1u : 0u;
        x.n_tiles = (uint32_t)((q.n + points - 1) / points);
    };
    tiles_of((int64_t)1 << p.tile_bits, 1, p.tile_bits);
    if (x.n_tiles < 0.84 * (double)(rounds * compute_units)) {   // the last round leaves many units without work: about as many tiles as there is room for
        const int64_t want = std::min<int64_t>(most, (q.n + rounds * compute_units - 1) / (rounds * compute_units));
        int shift = 0;
        while ((want + ((int64_t)1 << shift) - 1) >> shift > 255) ++shift;
        const int64_t factor = (want + ((int64_t)1 << shift) - 1) >> shift;
        if (factor << shift <= most) tiles_of(factor << shift, (uint32_t)factor, shift);
    }
    x.use = p.sorted && !runs_sparse(q, compute_units) && 2 * runs_lds_bytes(q.s, x.n_tiles) <= kMaxLdsBytes && !(q.far && q.n > 256 * most);
    const double run = (double)runs_block_edges(q.s) * (q.s + 1) / x.n_tiles;
    x.sums_lanes = q.grouped ? 32 : run < 12 ? 8 : run < 22 ? 16 : 32;
    return x;
}

// Mean-field sums by interpolation (field_kernels.h) or cell by cell (k_mean_field).
//   field_may, before anything is known of the embedding: enough work, and few cells in the heads' own groups, which are summed one by one either way.
//   field_pays, on the device, from the squares that have heads: us, 1.4e-4 a square and cell (256 nodes), 4.5e-5 a head (three polynomials of 256 terms, the place of the head
//   in its square's list) and 28 of launches against 2.45e-7 a cell and head, with a tenth to spare.  Mean-field sums, cell by cell -> field, us: 6 M x 1,638 in one square 2,364 -> 283, in
//   1,290 2,356 -> 593; 1 M x 2,000 in 460 518 -> 194; 500 k x 1,050 in one 142 -> 60, in 275 142 -> 101; 250 k x 2,100 in 221 156 -> 117.  Trained embeddings lie close: 6 M points in 1,638
//   clusters after 200 epochs within 10 of the origin.  An embedding it cannot use (looked at and left): 500 k x 1,050 145 -> 173.
//   field_sound: whether interpolation is as exact as float32, whatever the place of a head.  heaviest: the mass of the heaviest group; diameter: the largest distance
//   of a head and a cell.  The interpolant is off by up to kFieldError of a head's own group's mass, and what is left when that group is taken out is, in magnitudes,
//   at least D / (1 + D^2)^2 of the others' mass; the error may be 2^-24 of that.  Half of the mass in one group: extents up to 31; nine tenths: 15; a tenth: 64; a
//   twenty-fourth and less: any (62 sqrt 2 is the widest).  Nothing that is no number passes.
constexpr int kFieldMost = 2560;        // squares that can have heads
constexpr double kFieldEdge = 0.625;    // their sides
constexpr double kFieldError = 2e-12;   // of B; 1.5e-12 for the worst place of cell and head (A: 3.3e-13)
NOMAD_HOST_DEVICE inline bool field_sound(double heaviest, double diameter) {
    const double t = 1.0 + diameter * diameter;
    return kFieldError * heaviest <= 0x1p-24 * (1.0 - heaviest) * (diameter / (t * t));
}
inline bool field_may(double heads, double cells, double own_cells_of_all_heads, double heaviest) {
    return field_sound(heaviest, 2.0 * kFieldEdge) && cells >= 256 && heads * cells >= 5e8 && own_cells_of_all_heads <= heads * cells / 16;
}
NOMAD_HOST_DEVICE inline bool field_pays(double heads, double cells, double squares) {
    return squares <= kFieldMost && 1.4e-4 * squares * cells + 4.5e-5 * heads + 28.0 <= 0.9 * 2.45e-7 * heads * cells;
}

}  // namespace nomad
