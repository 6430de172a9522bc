// Device kernels of the edge pass for small embeddings: every workgroup holds 64-bit fixed-point sums of all points in LDS, so a
// force is two LDS additions and no record is made; the workgroups' sums are written side by side and added by a second kernel,
// which takes the step.
//
// What bounds an epoch of a few thousand points is the two kernels' chains of dependent steps.  With records those were a sort of the
// round (four barriers), chains of chunks and their walk: 9.3 + 10.0 us at 2,000 points and 46,734 positions; now 6.3 + 4.6, the memory's
// latency three times over, 400 vector instructions an edge and the sums' way out and back.  Same lanes for the same edges as
// k_edges_binned, same products, integer sums: the same bits.  (Rows fetched a round ahead: 8.4 us for one round, and no faster for
// several; 512 lanes: 6.1 us, but twice the sums.)
#pragma once
#include "nomad_kernels.h"

namespace nomad {

struct SmallArgs {
    const int32_t* head;          // [E] head of every CSR position
    unsigned long long* sums;     // [workgroups][x n, y n]
    float2* ghead;                // head sums of rows that lie inside one wavefront
    int64_t e_begin, e_end;       // CSR positions of this launch
};

template <int S, int KIND>
__global__ void __launch_bounds__(kSmallLanes) k_edges_small(const EdgeArgs args, const SmallArgs X) {
    constexpr int BS = kSmallLanes;
    EdgeArgs P = args;
    P.pool_size = 0; P.cS = nullptr; P.far = KIND == kFarEdges;
    if (KIND == kPlainEdges) P.group_of_cluster = nullptr;
    else __builtin_assume(P.group_of_cluster != nullptr);
    if (KIND == kGroupedEdges) P.gmembers = nullptr;
    extern __shared__ ulonglong2 lds_sums[];   // [x n, y n]
    unsigned long long* const sums = (unsigned long long*)lds_sums;
    const int tid = threadIdx.x;
    const uint32_t n = (uint32_t)P.n;
    BinArgs Q{};
    Q.ghead = X.ghead;
    int64_t e64 = X.e_begin + (int64_t)blockIdx.x * BS + tid;
    const int64_t stride = (int64_t)gridDim.x * BS;
    const auto position = [&](int64_t e) { return min(e, X.e_end - 1); };
    int32_t i = X.head[position(e64)], j = P.col[position(e64)];
    for (uint32_t l = tid; l < n; l += BS) lds_sums[l] = make_ulonglong2(0ull, 0ull);
    lds_barrier();
    for (int64_t e0 = e64 - tid; e0 < X.e_end; e0 += stride, e64 += stride) {
        EdgeFetch<S> f;
        float4 hi = make_float4(0.f, 0.f, 0.f, 0.f);
        if (P.group_of_cluster) hi = P.hinfo[i];
        issue_edge<S>(P, e64 < X.e_end, (int32_t)position(e64), i, j, hi, false, f);
        i = X.head[position(e64 + stride)];
        j = P.col[position(e64 + stride)];
        float hx = 0.f, hy = 0.f;
        const auto add = [&](uint32_t pt, float x, float y) {
            atomicAdd(sums + pt, to_fixed(x));
            atomicAdd(sums + n + pt, to_fixed(y));
        };
        if (f.has) {
            const HeadCtx h = head_of_fetch(P, f);
            if (P.far) resolve_far_negatives<S>(P, h.group, f);
            EdgeOut<(S > 0 ? S : 1)> o;
            edge_math<S, false>(h, P.pe ? f.pe : h.inv_deg, f.tj, f.tm, o);
            hx = o.hx;
            hy = o.hy;
            add((uint32_t)f.j, -o.a * o.dx, -o.a * o.dy);
#pragma unroll
            for (int k = 0; k < S; ++k)
                if (f.m[k] >= 0) add((uint32_t)f.m[k], o.rx[k], o.ry[k]);
        }
        if (reduce_head_sums(Q, f.has, f.i, f.row.x, f.row.y, e64, X.e_end, hx, hy)) add((uint32_t)f.i, hx, hy);
    }
    lds_barrier();
    ulonglong2* const out = (ulonglong2*)(X.sums + (size_t)blockIdx.x * 2 * n);
    for (uint32_t l = tid; l < n; l += BS) out[l] = lds_sums[l];
}

// Adds the workgroups' sums of 32 points (256 lanes: 64 sums in four parts), then what finish_tile does.
__global__ void __launch_bounds__(256) k_small_finish(const unsigned long long* __restrict__ sums, uint32_t n_wg, float2* __restrict__ ghead, float2* __restrict__ g,
                                                      uint32_t n, float2* __restrict__ theta, float eta) {
    __shared__ unsigned long long acc[4][64];   // x of 32 points, then y
    const uint32_t p0 = blockIdx.x * 32u, c = threadIdx.x & 63u, part = threadIdx.x >> 6;
    const uint32_t pt = min(p0 + (c & 31u), n - 1u), at = c < 32u ? pt : n + pt;
    const float2 hd = ghead[pt], t = theta[pt];   // (used by the first 32 lanes)
    unsigned long long s = 0ull;
    uint32_t w = part;
    for (; w + 28u < n_wg; w += 32u) {
        unsigned long long v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = sums[(size_t)(w + 4u * u) * 2 * n + at];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; w < n_wg; w += 4u) s += sums[(size_t)w * 2 * n + at];
    acc[part][c] = s;
    __syncthreads();
    if (threadIdx.x >= 32u || p0 + threadIdx.x >= n) return;
    const uint32_t l = threadIdx.x;
    const float2 gi = point_gradient(hd, acc[0][l] + acc[1][l] + acc[2][l] + acc[3][l], acc[0][32 + l] + acc[1][32 + l] + acc[2][32 + l] + acc[3][32 + l]);
    ghead[pt] = make_float2(0.f, 0.f);
    g[pt] = gi;
    theta[pt] = stepped(t, gi, eta);
}

}  // namespace nomad
