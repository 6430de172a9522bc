// Device kernels of the exchanged edge pass: the rows an edge needs are brought to it, and the forces it makes are taken
// away, tile by tile through memory, so that nothing is gathered from or scattered to random addresses.
//
// The sorted edge pass (k_edges_binned) gathers theta_m of every negative from anywhere in the embedding.  Once the embedding is
// larger than the L2s a gather costs a line of 128 bytes for its 8, and the rate of such lines bounds the epoch whatever the
// kernel does.  Here a block of EB consecutive CSR positions deals its (s + 1) references per edge (tail, negatives)
// to the tiles they point into, which needs no embedding at all; the tiles, with their rows in LDS, answer every reference;
// the edge pass then reads its block's answers as one run, and writes the forces over them; the tiles collect those.  A
// reference keeps one slot of its block through all four kernels:
//
//   k_exchange_deal   draws the negatives, counting-sorts the block's references by tile in LDS: idx[slot] = low bits of the point
//                     (16 bits, written as one run), pos[edge][k] = slot (16 bits), runs[block][tile] = first slot and length
//   k_exchange_rows   one workgroup per tile or pair of tiles (and part of the blocks): rec[slot] = theta of the point, from LDS
//   k_exchange_edges  the block's answers to LDS (one run), the arithmetic of its edges, forces back to their slots, the
//                     block written back (one run); head sums as in k_edges_binned
//   k_tile_sums       one workgroup per tile: forces into 64-bit fixed-point sums in LDS, then the step (finish_tile)
//
// Same lanes for the same edges as k_edges_binned, same products, integer sums: the same bits.
//
// A reference costs 42 bytes in streams (2 + 2 out, 2 in and 8 out, 10 in and 8 out, 10 in) where the sorted pass fetches a line of
// 128 and moves 24.  Ten million points, 3.0e8 positions, s = 5, a quarter of the epoch's positions a launch: edge pass 9.2 ms and
// tile pass 1.1 before; deal 0.66 (vector pipe and LDS counters), rows 2.49, edges 1.82 (5.0 TB/s: a copy's rate), sums 2.15; the
// epoch 41.3 -> 28.7 ms.  A million points, directed: 1.33 -> 1.15 ms an epoch.  What holds rows and sums is the short run:
// without its stores k_exchange_rows takes 0.6 of 2.1 ms, and pieces of 120 bytes at any 8-byte boundary are written at 1.7 TB/s
// where whole 64-byte sectors go at 3.4 and a stream at 5.4.  Tried: answers laid out tile by tile, staged in LDS and written in whole
// sectors, read piecewise by the edges (rows 2.4, but its short reads then fetch 7.2 GB for 1.4; edges 2.06); non-temporal
// stores (2.9); more loads in flight a wavefront or two steps ahead (the same).
#pragma once
#include "nomad_kernels.h"

namespace nomad {

struct ExchangeArgs {
    const int32_t* head;     // [E] head of every CSR position
    float2* rec;             // [blocks][slots] rows on their way to the edges, then forces on their way to the points
    uint16_t* idx;           // [blocks][slots] low bits of the point
    uint32_t* pos;           // [blocks][(s + 2) / 2][EB] slots of an edge's references, two to a word
    uint16_t* side;          // [blocks][EB / 64][2] slots of the partial head sums a wavefront hands on
    uint32_t* runs;          // [blocks][tiles] first slot | length << 16
    float2* ghead;           // head sums of rows that lie inside one wavefront
    int64_t e_begin, e_end;  // CSR positions of this launch
    uint32_t n_blocks, n_tiles;
    int tile_bits;
    uint32_t spare;          // first of the kExchangeSpare slots behind the last block's
    uint32_t points, magic;  // k_edges_runs: points of a tile, runs_tile_of's numbers
    int shift;
};

template <int S>
struct ExchangeShape {
    static constexpr int R = exchange_edges_per_lane(S);              // edges per lane
    static constexpr int EB = kExchangeLanes * R;                      // edges per block
    static constexpr int SLOTS = (int)exchange_slots(S);               // slots of a block, padded
    static constexpr int PAIRS = (S + 2) / 2;
    static constexpr int WAVES = EB / 64;
};

// whether the lane holds the last edge of a row inside its wavefront, and whether that row lies inside it (reduce_head_sums)
__device__ __forceinline__ bool hands_on_head_sum(bool has, int32_t ea, int32_t eb, int64_t e64, int64_t e_end) {
    const int lane = threadIdx.x & 63;
    const int64_t wave_e0 = e64 - lane;
    const bool row_end = has && (lane == 63 || e64 + 1 >= min((int64_t)eb, e_end));
    const bool inside = (int64_t)ea >= wave_e0 && (int64_t)eb <= min(wave_e0 + 64, e_end);
    return row_end && !inside;
}

// The references that a block has for every tile (`first`, in LDS, complete) become their first slots there, and the block's table of runs; all BS lanes call.  Returns
// how many there are.
template <int BS>
__device__ __forceinline__ uint32_t counts_to_runs(uint32_t* first, uint32_t T, uint32_t (&wave_total)[BS / 64], uint32_t* __restrict__ runs) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t per = (T + BS - 1) / BS, b0 = (uint32_t)tid * per;
    uint32_t own = 0;
    for (uint32_t x = 0; x < per; ++x) own += b0 + x < T ? first[b0 + x] : 0u;
    const uint32_t incl = wave_prefix(own);
    if (lane == 63) wave_total[wave] = incl;
    lds_barrier();
    const uint32_t waves_incl = wave_prefix(lane < BS / 64 ? wave_total[lane] : 0u);
    uint32_t run = incl - own;
    if (wave > 0) run += (uint32_t)__builtin_amdgcn_readlane((int)waves_incl, wave - 1);
    for (uint32_t x = 0; x < per; ++x)
        if (b0 + x < T) {
            const uint32_t c = first[b0 + x];
            first[b0 + x] = run;
            runs[b0 + x] = run | c << 16;
            run += c;
        }
    return (uint32_t)__builtin_amdgcn_readlane((int)waves_incl, BS / 64 - 1);
}

template <int S>
__global__ void __launch_bounds__(kExchangeLanes) k_exchange_deal(const EdgeArgs args, const ExchangeArgs X) {
    using Shape = ExchangeShape<S>;
    constexpr int R = Shape::R, BS = kExchangeLanes;
    EdgeArgs P = args;
    P.pool_size = 0;
    P.group_of_cluster = nullptr;
    extern __shared__ uint32_t lds_deal[];
    uint16_t* const pts = (uint16_t*)lds_deal;                      // [SLOTS] the block's references in slot order
    uint32_t* const first = lds_deal + Shape::SLOTS / 2;            // [tiles] count, then first slot
    __shared__ uint32_t wave_total[BS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t blk = blockIdx.x, T = X.n_tiles;
    const int tb = X.tile_bits;
    const int64_t e0 = X.e_begin + (int64_t)blk * Shape::EB;
    int32_t i[R], j[R];
    RowBounds row[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t e = min(e0 + r * BS + tid, X.e_end - 1);
        i[r] = X.head[e];
        j[r] = P.col[e];
    }
    for (uint32_t b = tid; b < T; b += BS) first[b] = 0u;
    const Population all = {0u, (uint32_t)P.n, nullptr};
    uint32_t pt[R][S + 2], rank[R][S + 2];
    bool has[R], hands_on[R];
#pragma unroll
    for (int r = 0; r < R; ++r) row[r] = *(const RowBounds*)(P.row_ptr + i[r]);
    lds_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t e = e0 + r * BS + tid;
        has[r] = e < X.e_end;
        hands_on[r] = hands_on_head_sum(has[r], row[r].x, row[r].y, e, X.e_end);
        int32_t m[S > 0 ? S : 1];
        draw_negatives<S>(P, all, (int32_t)min(e, X.e_end - 1), m);
#pragma unroll
        for (int k = 0; k < S; ++k) pt[r][k + 1] = (uint32_t)m[k];
        pt[r][0] = (uint32_t)j[r];
        pt[r][S + 1] = (uint32_t)i[r];
#pragma unroll
        for (int k = 0; k < S + 2; ++k) {
            rank[r][k] = 0u;
            if (k <= S ? has[r] : hands_on[r]) rank[r][k] = atomicAdd(&first[pt[r][k] >> tb], 1u);
        }
    }
    lds_barrier();
    counts_to_runs<BS>(first, T, wave_total, X.runs + (size_t)blk * T);
    lds_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t at[S + 2];
#pragma unroll
        for (int k = 0; k < S + 2; ++k) {
            at[k] = 0u;
            if (k <= S ? has[r] : hands_on[r]) {
                at[k] = first[pt[r][k] >> tb] + rank[r][k];
                pts[at[k]] = (uint16_t)pt[r][k];
            }
        }
#pragma unroll
        for (int p = 0; p < Shape::PAIRS; ++p)
            X.pos[((size_t)blk * Shape::PAIRS + p) * Shape::EB + r * BS + tid] = at[2 * p] | (2 * p + 1 <= S ? at[2 * p + 1] << 16 : 0u);
        if (hands_on[r]) {
            const int w = r * (BS / 64) + wave;
            const bool left = (int64_t)row[r].x < e0 + r * BS + wave * 64;   // the row began before this wavefront's positions
            X.side[((size_t)blk * Shape::WAVES + w) * 2 + (left ? 0 : 1)] = (uint16_t)at[S + 1];
        }
    }
    lds_barrier();
    uint4* const out = (uint4*)(X.idx + (size_t)blk * Shape::SLOTS);
    for (int u = tid; u < Shape::SLOTS / 8; u += BS) out[u] = ((const uint4*)pts)[u];
}

// Walks the references of tile b in the blocks blk0 .. blk1-1, the whole workgroup side by side: G lanes take the first G
// references of one block's run, U runs each a step, and the next G of all U where some run has more; what a run has beyond 2 G a
// whole wavefront takes, one run after the other, each a wait for memory of its own.  (With everything beyond G taken that way the
// mean run must not be about as long as there are lanes: 1,060,000 points in random order, runs of 71 on 64 lanes, 1.52 ms an epoch on
// the sorted pass, 1.66 on the exchange, now 1.27; s = 3 1.08, 1.13, 0.90.)  The runs' bounds are read
// a step before their references are loaded, and those AHEAD steps before they are used: memory operations of a wavefront end in
// order, so a load is waited for together with the stores before it.
//   load(slot) -> T; use(T, whether the lane has a reference)
// Loads and uses are straight-line code (a lane without a reference takes its run's first, or a slot behind the last block's that
// means nothing): behind a branch every load would be waited for by itself.  All lanes must call.
template <int BS, int G, int U, int AHEAD, bool PAIR, typename T, typename Load, typename Use>
__device__ __forceinline__ void walk_tile_runs(const ExchangeArgs& X, uint32_t b, uint32_t slots, uint32_t blk0, uint32_t blk1, Load load, Use use) {
    static_assert(U <= G, "one lane of the group holds the bounds of one run");
    constexpr uint32_t RW = BS / G, STEP = RW * U;      // runs side by side, runs a step
    constexpr int BUF = AHEAD + 1;
    const uint32_t lane = threadIdx.x & 63u, k = threadIdx.x % G, group = threadIdx.x / G;
    const uint32_t nowhere = X.spare + ((blockIdx.x * 64u + lane) & (kExchangeSpare - 1u));
    struct Bounds { uint32_t first, len; };
    const auto bounds = [&](uint32_t q0) {
        const uint32_t q = q0 + (k % U) * RW + group, have = min(q, blk1 - 1u);
        const uint32_t* const e = X.runs + (size_t)have * X.n_tiles + b;
        Bounds r;
        r.first = have * slots + (e[0] & 0xFFFFu);
        r.len = e[0] >> 16;
        if (PAIR && b + 1 < X.n_tiles) r.len += e[1] >> 16;   // (a pair of tiles: their runs are neighbours)
        if (q >= blk1) r.len = 0u;
        return r;
    };
    T v[BUF][U];
    uint32_t has[BUF];   // a bit per reference
    const auto fetch = [&](const Bounds& r, T (&d)[U], uint32_t& h) {
        h = 0u;
        uint32_t first[U], len[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int src = (int)((lane & ~(uint32_t)(G - 1)) + u);
            first[u] = (uint32_t)__shfl((int)r.first, src, 64);
            len[u] = (uint32_t)__shfl((int)r.len, src, 64);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = len[u] > k;
            d[u] = load(len[u] ? first[u] + (in ? k : 0u) : nowhere);
            h |= in ? 1u << u : 0u;
        }
        if (!__any(k < (uint32_t)U && r.len > (uint32_t)G)) return;
        {   // the next G of the runs that have more
            T dd[U];
#pragma unroll
            for (int u = 0; u < U; ++u) dd[u] = load(len[u] ? first[u] + (len[u] > G + k ? G + k : 0u) : nowhere);
#pragma unroll
            for (int u = 0; u < U; ++u) use(dd[u], len[u] > G + k);
        }
        unsigned long long which = __ballot(k < (uint32_t)U && r.len > 2u * G);
        while (which) {
            const int src = __ffsll((long long)which) - 1;
            which &= which - 1ull;
            const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)r.first, src), n = (uint32_t)__builtin_amdgcn_readlane((int)r.len, src);
            constexpr int V = 4;
            for (uint32_t p = 2 * G + lane; p - lane < n; p += 64 * V) {
                T dd[V];
#pragma unroll
                for (int x = 0; x < V; ++x) dd[x] = load(from + min(p + x * 64u, n - 1u));
#pragma unroll
                for (int x = 0; x < V; ++x) use(dd[x], p + x * 64u < n);
            }
        }
    };
    const auto consume = [&](const T (&d)[U], uint32_t h) {
#pragma unroll
        for (int u = 0; u < U; ++u) use(d[u], (h >> u & 1u) != 0u);
    };
    Bounds next = bounds(blk0);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
        const Bounds r = next;
        next = bounds(blk0 + (i + 1) * STEP);
        fetch(r, v[i], has[i]);
    }
    for (uint32_t q0 = blk0; q0 < blk1; q0 += BUF * STEP)
#pragma unroll
        for (int i = 0; i < BUF; ++i) {   // step q0 + i * STEP is used, the one AHEAD of it is fetched (past the end: nothing)
            constexpr int A = AHEAD;
            const Bounds r = next;
            next = bounds(q0 + (i + A + 1) * STEP);
            fetch(r, v[(i + A) % BUF], has[(i + A) % BUF]);
            consume(v[i], has[i]);
        }
}

// The tile (and part) of a workgroup: workgroups go to the 8 XCDs round-robin, and kExchangeTilesTogether neighbouring tiles go to
// one XCD, so that their adjacent runs are read and written through one L2; the next ones to the next XCD, because the tails of a
// launch's positions lie in a stretch of the tiles (an eighth of the tiles each: 1.4 times as long at ten million points).
__device__ __forceinline__ bool exchange_unit(uint32_t n_tiles, uint32_t& tile, uint32_t& part) {
    const uint32_t padded = exchange_padded_tiles(n_tiles), v = blockIdx.x % padded, x = v & 7u, y = v >> 3;
    part = blockIdx.x / padded;
    tile = (y / kExchangeTilesTogether * 8u + x) * kExchangeTilesTogether + y % kExchangeTilesTogether;
    return tile < n_tiles;
}

template <int G, bool PAIR>
__global__ void __launch_bounds__(1024) k_exchange_rows(const ExchangeArgs X, const float2* __restrict__ theta, int64_t n, uint32_t slots, uint32_t parts) {
    extern __shared__ float2 lds_rows[];
    uint32_t b, part;
    if (!exchange_unit(PAIR ? (X.n_tiles + 1) / 2 : X.n_tiles, b, part)) return;
    if (PAIR) b *= 2;
    const int64_t p0 = (int64_t)b << X.tile_bits;
    const uint32_t mask = ((PAIR ? 2u : 1u) << X.tile_bits) - 1u;
    const int tile = (int)min((int64_t)mask + 1, n - p0);
    for (int l = threadIdx.x; l < tile; l += 1024) lds_rows[l] = theta[p0 + l];
    __syncthreads();
    const uint32_t q0 = (uint32_t)((uint64_t)X.n_blocks * part / parts), q1 = (uint32_t)((uint64_t)X.n_blocks * (part + 1) / parts);
    if (q0 >= q1) return;
    // a lane without a reference writes its run's first row once more, or into the spare slots
    struct Ref { uint32_t at; uint16_t l; };
    walk_tile_runs<1024, G, 8, 1, PAIR, Ref>(X, b, slots, q0, q1, [&](uint32_t at) { return Ref{at, X.idx[at]}; },
                                                    [&](const Ref& v, bool) { X.rec[v.at] = lds_rows[v.l & mask]; });
}

// Two workgroups per compute unit: one loads or writes while the other computes.
template <int S>
__global__ void __launch_bounds__(kExchangeLanes) k_exchange_edges(const EdgeArgs args, const ExchangeArgs X) {
    using Shape = ExchangeShape<S>;
    constexpr int R = Shape::R, BS = kExchangeLanes;
    EdgeArgs P = args;
    P.pool_size = 0; P.cS = nullptr; P.far = 0; P.group_of_cluster = nullptr;
    extern __shared__ float2 lds_rec[];   // [SLOTS]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t blk = blockIdx.x;
    const int64_t e0 = X.e_begin + (int64_t)blk * Shape::EB;
    float4* const rec = (float4*)(X.rec + (size_t)blk * Shape::SLOTS);
    constexpr int HALF = Shape::SLOTS / 2, LOADS = (HALF + BS - 1) / BS;   // float4 of a block
    EdgeFetch<S> f[R];
    uint32_t pos[R][Shape::PAIRS], side[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t e = e0 + r * BS + tid, c = min(e, X.e_end - 1);
        f[r].has = e < X.e_end;
        f[r].i = X.head[c];
        if (P.pe) f[r].pe = P.pe[c];
    }
    float4 in[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) in[u] = rec[min(u * BS + tid, HALF - 1)];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int p = 0; p < Shape::PAIRS; ++p) pos[r][p] = X.pos[((size_t)blk * Shape::PAIRS + p) * Shape::EB + r * BS + tid];
        side[r] = X.side[((size_t)blk * Shape::WAVES + r * (BS / 64) + wave) * 2 + (lane & 1)];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        f[r].row = *(const RowBounds*)(P.row_ptr + f[r].i);
        f[r].ti = P.theta[f[r].i];
    }
#pragma unroll
    for (int u = 0; u < LOADS; ++u)
        if (u * BS + tid < HALF) ((float4*)lds_rec)[u * BS + tid] = in[u];
    lds_barrier();
    BinArgs Q{};
    Q.ghead = X.ghead;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t e64 = e0 + r * BS + tid;
        float hx = 0.f, hy = 0.f;
        if (f[r].has) {
            uint32_t slot[S + 1];
#pragma unroll
            for (int k = 0; k <= S; ++k) slot[k] = k & 1 ? pos[r][k / 2] >> 16 : pos[r][k / 2] & 0xFFFFu;
            f[r].tj = lds_rec[slot[0]];
#pragma unroll
            for (int k = 0; k < S; ++k) f[r].tm[k] = lds_rec[slot[k + 1]];
            const HeadCtx h = head_of_fetch(P, f[r]);
            EdgeOut<(S > 0 ? S : 1)> o;
            edge_math<S, false>(h, P.pe ? f[r].pe : h.inv_deg, f[r].tj, f[r].tm, o);
            hx = o.hx;
            hy = o.hy;
            lds_rec[slot[0]] = make_float2(-o.a * o.dx, -o.a * o.dy);
#pragma unroll
            for (int k = 0; k < S; ++k) lds_rec[slot[k + 1]] = make_float2(o.rx[k], o.ry[k]);
        }
        const uint32_t side_left = (uint32_t)__builtin_amdgcn_readlane((int)side[r], 0), side_right = (uint32_t)__builtin_amdgcn_readlane((int)side[r], 1);
        if (reduce_head_sums(Q, f[r].has, f[r].i, f[r].row.x, f[r].row.y, e64, X.e_end, hx, hy))
            lds_rec[(int64_t)f[r].row.x < e64 - lane ? side_left : side_right] = make_float2(hx, hy);
    }
    lds_barrier();
    for (int u = tid; u < HALF; u += BS) rec[u] = ((const float4*)lds_rec)[u];
}

// What the sums need to know of the edge pass that made the forces.
struct TileSums {
    const float2* rec;       // [blocks][slots] forces, a block's in the order of the tiles
    const uint16_t* idx;     // [blocks][slots] point inside the tile, under the mask
    const uint32_t* runs;    // [blocks][tiles] first slot | length << 16
    float2* ghead;           // head sums of rows that lie inside one wavefront
    uint32_t n_blocks, slots, n_tiles, points, mask;
    uint32_t spare;          // first of the kExchangeSpare slots behind the last block's
};

// Adds the forces of a tile into 64-bit fixed-point sums in LDS, then what finish_tile does.
//
// What bounds it is the handling of short runs, not the additions: with a load a reference and lanes that wait for the longest of the runs
// beside theirs, 90 M references in runs of 37 took 288 us.  Here a wavefront reads the runs of its share of the blocks, 64 at a time, and
// queues what is not empty in LDS as segments of up to 2 G references (a long run is several); a step takes 64 / G segments, two
// references a lane, and its loads are under way while the step before is added.  Two steps are written out one after the other, so that
// no copy of what is under way is made, which would wait for it: 288 -> 268 us; 450 M references in runs of 7.5 2.27 -> 2.15 ms.
// (Runs that begin at even slots, for aligned loads: no difference.  Two segments a lane and step: the same, at half as many registers again.)
template <int G>
__global__ void __launch_bounds__(kBinBlock) k_tile_sums(const TileSums X, float2* __restrict__ g, int64_t n, float2* __restrict__ theta, float eta,
                                                        unsigned long long* __restrict__ carry, int phase) {
    constexpr uint32_t STEP = 64 / G, WAVES = kBinBlock / 64, SPAN = 64u * WAVES;   // segments a step; blocks the workgroup reads the runs of at once
    typedef float Forces __attribute__((ext_vector_type(4), aligned(8)));
    typedef uint32_t Indexes __attribute__((aligned(2)));
    extern __shared__ unsigned long long acc[];   // [2 tile]: x, then y
    __shared__ uint2 queues[WAVES][tile_sums_queue(G)];
    uint32_t b, part;
    if (!exchange_unit(X.n_tiles, b, part)) return;
    const uint32_t blocks = X.n_blocks, mask = X.mask;
    const int tile = (int)X.points;
    for (int l = threadIdx.x; l < 2 * tile; l += kBinBlock) acc[l] = 0ull;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), k2 = 2u * (lane % G), group = lane / G;
    const uint32_t nowhere = X.spare + ((b * 128u + 2u * lane) & (kExchangeSpare - 1u));   // (an even slot of the spare ones: two can be read there)
    uint2* const queue = queues[wave];
    uint32_t count = 0;   // segments queued: first slot, references
    struct Two { Forces f; uint32_t l, len; };
    // this lane's references of the segments from .. from + STEP-1 of the queue, of which there are `have`
    const auto fetch = [&](Two& d, uint32_t from, uint32_t have) {
        const uint2 seg = queue[from + group];
        d.len = group < have ? seg.y : 0u;
        const uint32_t at = d.len > k2 ? seg.x + k2 : nowhere;
        d.f = *(const Forces*)(X.rec + at);
        d.l = *(const Indexes*)(X.idx + at);
    };
    const auto add = [&](uint32_t l, float x, float y) {
        atomicAdd(&acc[l], to_fixed(x));
        atomicAdd(&acc[tile + l], to_fixed(y));
    };
    const auto consume = [&](const Two& d) {
        if (k2 < d.len) add(d.l & mask, d.f.x, d.f.y);
        if (k2 + 1u < d.len) add(d.l >> 16 & mask, d.f.z, d.f.w);
    };
    Two v0 = {0.f, 0u, 0u}, v1;
    const auto two_steps = [&](uint32_t have) {
        fetch(v1, count, have);
        consume(v0);
        fetch(v0, count + STEP, max(have, STEP) - STEP);
        consume(v1);
    };
    const auto run_of = [&](uint32_t q0) {   // neighbouring blocks go to different wavefronts
        const uint32_t q = q0 + lane * WAVES + wave, have = min(q, blocks - 1u), e = X.runs[(size_t)have * X.n_tiles + b];
        return make_uint2(have * X.slots + (e & 0xFFFFu), q < blocks ? e >> 16 : 0u);
    };
    uint2 next = run_of(0u);
    for (uint32_t q0 = 0; q0 < blocks; q0 += SPAN) {
        uint2 run = next;
        next = run_of(q0 + SPAN);
        unsigned long long some;
        while ((some = __ballot(run.y != 0u)) != 0ull) {
            const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
            if (run.y) queue[count + before] = make_uint2(run.x, min(run.y, 2u * G));
            run.x += 2u * G;
            run.y -= min(run.y, 2u * G);
            count += (uint32_t)__popcll(some);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");   // (the queue is the wavefront's own)
            while (count >= 2u * STEP) {
                count -= 2u * STEP;
                two_steps(2u * STEP);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        }
    }
    const uint32_t left = count;
    count = 0u;
    two_steps(left);
    consume(v0);
    __syncthreads();
    finish_tile(acc, (int64_t)b * tile, tile, X.ghead, g, n, theta, eta, nullptr, nullptr, carry, phase);
}

}  // namespace nomad
