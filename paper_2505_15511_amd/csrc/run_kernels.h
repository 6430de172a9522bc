// Device kernel of the edge pass that gathers the rows it needs and leaves its forces in runs, a block's by tile, for k_tile_sums
// (exchange_kernels.h) to collect: embeddings whose rows are mostly in the L2s.
#pragma once
#include "exchange_kernels.h"

namespace nomad {

template <int S>
struct RunsShape {
    static constexpr int BS = runs_lanes(S), R = runs_edges_per_lane(S), EB = runs_block_edges(S);
    static constexpr int SLOTS = (int)runs_slots(S);
};

// A block of EB consecutive CSR positions a workgroup: gathers, ranks of the references in their tiles (LDS counters, while the gathers
// are under way), first slots, the arithmetic of the edges, forces and points to their slots in LDS, both out as one stretch.
//
// Bound by the gathers out of L2 (2.6 M edges of 100,000 points, s = 5: 78 us, the 15.6 M gathers alone 58 at 270 G/s).  k_edges_binned does the same work in 141 us:
// one persistent workgroup a compute unit, whose rounds are a chain of phases with barriers between them, and records of 12 bytes in chains of chunks.  Here a
// compute unit has two workgroups of 1,024 lanes (s = 7 and 8: three of 512; up to two negatives two of 512 with three edges a lane), each in a phase of its own, a block's forces leave as whole lines, 10 bytes a reference,
// and the tile's workgroup finds its runs by a table (the tile pass 54 -> 36 us).  300,000 points, 9 M edges: 285 + 165 us.  6 M points in groups, s = 2: 3.92 + 0.94 -> 2.74 + 1.02 ms.
// Same lanes for the same edges, same products, integer sums: the same bits.
template <int S, int KIND>
__global__ void __launch_bounds__(runs_lanes(S), runs_waves_per_simd(S)) k_edges_runs(const EdgeArgs args, const ExchangeArgs X) {
    using Shape = RunsShape<S>;
    constexpr int R = Shape::R, BS = Shape::BS;
    EdgeArgs P = args;
    P.pool_size = 0; P.cS = nullptr; P.far = KIND == kFarEdges;
    if (KIND == kPlainEdges) P.group_of_cluster = nullptr;
    else __builtin_assume(P.group_of_cluster != nullptr);
    P.gmembers = nullptr;
    extern __shared__ float2 lds_runs[];
    float2* const rec = lds_runs;                                     // [SLOTS] forces
    uint16_t* const pts = (uint16_t*)(lds_runs + Shape::SLOTS);       // [SLOTS] points
    uint32_t* const first = (uint32_t*)(pts + Shape::SLOTS);          // [tiles] references, then first slot
    __shared__ uint32_t wave_total[BS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t blk = blockIdx.x, T = X.n_tiles;
    const int64_t e0 = X.e_begin + (int64_t)blk * Shape::EB;
    EdgeFetch<S> f[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t e = e0 + r * BS + tid, c = min(e, X.e_end - 1);
        f[r].has = e < X.e_end;
        f[r].e = (int32_t)c;
        f[r].i = X.head[c];
        f[r].j = P.col[c];
        if (P.pe) f[r].pe = P.pe[c];
    }
    for (uint32_t b = tid; b < T; b += BS) first[b] = 0u;
    if (KIND != kPlainEdges) {
#pragma unroll
        for (int r = 0; r < R; ++r) f[r].hi = P.hinfo[f[r].i];
    }
    if (KIND != kGroupedEdges) {   // (of all points: nothing to wait for)
#pragma unroll
        for (int r = 0; r < R; ++r) draw_negatives<S>(P, Population{0u, (uint32_t)P.n, nullptr}, f[r].e, f[r].m);
    }
    // the bounds of the rows first: the ranks wait for them, and the gathers behind them stay under way
#pragma unroll
    for (int r = 0; r < R; ++r) f[r].row = *(const RowBounds*)(P.row_ptr + f[r].i);
    if (KIND == kGroupedEdges) {
#pragma unroll
        for (int r = 0; r < R; ++r) draw_negatives<S>(P, Population{__float_as_uint(f[r].hi.x), __float_as_uint(f[r].hi.y), nullptr}, f[r].e, f[r].m);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        f[r].ti = P.theta[f[r].i];
        f[r].tj = P.theta[f[r].j];
#pragma unroll
        for (int k = 0; k < S; ++k) f[r].tm[k] = KIND == kFarEdges ? make_float2(__int_as_float(P.cluster_of[f[r].m[k]]), 0.f) : P.theta[f[r].m[k]];
        if (KIND == kGroupedEdges) { f[r].A = P.A[f[r].i]; f[r].B = P.B[f[r].i]; }
    }
    if (KIND == kFarEdges) {
#pragma unroll
        for (int r = 0; r < R; ++r) resolve_far_negatives<S>(P, __float_as_int(f[r].hi.w), f[r]);
    }
    lds_barrier();
    const auto point = [&](int r, int k) { return (uint32_t)(k == 0 ? f[r].j : k <= S ? f[r].m[k > 0 && k <= S ? k - 1 : 0] : f[r].i); };
    uint32_t place[R][S + 2];   // tile | references of the block before it there << 16
    bool valid[R][S + 2];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool on = hands_on_head_sum(f[r].has, f[r].row.x, f[r].row.y, e0 + r * BS + tid, X.e_end);
#pragma unroll
        for (int k = 0; k < S + 2; ++k) {
            valid[r][k] = k > S ? on : f[r].has && (KIND != kFarEdges || k == 0 || f[r].m[k > 0 ? k - 1 : 0] >= 0);
            place[r][k] = 0u;
            if (valid[r][k]) {
                const uint32_t tile = runs_tile_of(point(r, k), X.shift, X.magic);
                place[r][k] = tile | atomicAdd(&first[tile], 1u) << 16;
            }
        }
    }
    lds_barrier();
    const uint32_t used = counts_to_runs<BS>(first, T, wave_total, X.runs + (size_t)blk * T);
    lds_barrier();
    BinArgs Q{};
    Q.ghead = X.ghead;
    const auto put = [&](uint32_t pt, uint32_t where, float x, float y) {
        const uint32_t tile = where & 0xFFFFu, at = first[tile] + (where >> 16);
        rec[at] = make_float2(x, y);
        pts[at] = (uint16_t)(pt - tile * X.points);
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float hx = 0.f, hy = 0.f;
        if (f[r].has) {
            const HeadCtx h = head_of_fetch(P, f[r]);
            EdgeOut<(S > 0 ? S : 1)> o;
            edge_math<S, false>(h, P.pe ? f[r].pe : h.inv_deg, f[r].tj, f[r].tm, o);
            hx = o.hx;
            hy = o.hy;
            put((uint32_t)f[r].j, place[r][0], -o.a * o.dx, -o.a * o.dy);
#pragma unroll
            for (int k = 0; k < S; ++k)
                if (KIND != kFarEdges || valid[r][k + 1]) put((uint32_t)f[r].m[k], place[r][k + 1], o.rx[k], o.ry[k]);
        }
        if (reduce_head_sums(Q, f[r].has, f[r].i, f[r].row.x, f[r].row.y, e0 + r * BS + tid, X.e_end, hx, hy)) put((uint32_t)f[r].i, place[r][S + 1], hx, hy);
    }
    lds_barrier();
    float4* const out_rec = (float4*)(X.rec + (size_t)blk * Shape::SLOTS);
    uint4* const out_idx = (uint4*)(X.idx + (size_t)blk * Shape::SLOTS);
    for (int u = tid; u < (int)((used + 1) / 2); u += BS) out_rec[u] = ((const float4*)rec)[u];
    for (int u = tid; u < (int)((used + 7) / 8); u += BS) out_idx[u] = ((const uint4*)pts)[u];
}

}  // namespace nomad
