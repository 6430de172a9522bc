// libnomad: the instances of the nearest-neighbour filter kernel and their launch (a source of its own: they are most of the
// index's compile time).
#include <type_traits>

#include "knn_filter.h"

namespace {

template <int TILE, int KS, int L, int WAVES, int WAY = kWaySift>
hipError_t launch(hipStream_t st, uint32_t n_blocks, const KnnSets& P, const KnnBlock* blocks, int32_t list_len, int32_t* cand, float* keys, float* tau,
                  const KnnAssign& assign) {
    constexpr size_t lds = knn_filter_lds_bytes(TILE, KS, L, WAVES, WAY == kWayAlone ? 1 : 2);
    static_assert(lds <= 160 * 1024, "");
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)k_knn_filter<TILE, KS, L, WAVES, WAY>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_knn_filter<TILE, KS, L, WAVES, WAY>), dim3(n_blocks), dim3(64 * WAVES), lds, st, P, blocks, list_len, cand, keys, tau, assign);
    return hipGetLastError();
}

// list classes: 0 = one neighbour, 1 = short lists, 2 = long ones
template <int TILE, int KS, int L>
hipError_t launch_waves(hipStream_t st, uint32_t n_blocks, int waves, const KnnSets& P, const KnnBlock* blocks, int32_t list_len, int32_t* cand,
                        float* keys, float* tau, const KnnAssign& assign) {
    constexpr int kMost = knn_most_waves(TILE, KS, L), kFew = TILE == 32 ? 2 : 4;
    if (kMost > 8 && waves == kMost) return launch<TILE, KS, L, kMost>(st, n_blocks, P, blocks, list_len, cand, keys, tau, assign);
    const auto way = [&](auto w) {
        if (waves == 8) return launch<TILE, KS, L, 8, decltype(w)::value>(st, n_blocks, P, blocks, list_len, cand, keys, tau, assign);
        return launch<TILE, KS, L, kFew, decltype(w)::value>(st, n_blocks, P, blocks, list_len, cand, keys, tau, assign);
    };
    if constexpr (knn_shares(TILE, KS, L))
        if (P.shared) return way(std::integral_constant<int, kWayShare>());
    if (P.shared) return hipErrorInvalidValue;   // (knn_shares: the caller asks)
    if constexpr (L > 2 && !knn_both_ways(TILE, KS, 8))
        if (!P.ordered) return way(std::integral_constant<int, kWayBeside>());
    if constexpr (L == 2)
        if (P.alone) return waves == 8 ? launch<TILE, KS, L, 8, kWayAlone>(st, n_blocks, P, blocks, list_len, cand, keys, tau, assign) : hipErrorInvalidValue;   // (products_may_be_alone)
    return way(std::integral_constant<int, kWaySift>());
}

}  // namespace

#define NOMAD_ARGS st, n_blocks, waves, P, blocks, list_len, cand, keys, tau, assign
hipError_t launch_knn_filter(hipStream_t st, uint32_t n_blocks, int waves, const KnnSets& P, const KnnBlock* blocks, int32_t list_len,
                             int32_t* cand, float* keys, float* tau, const KnnAssign& assign) {
    if (n_blocks == 0) return hipSuccess;
    const int tile = knn_tile(P.d, list_len), steps = knn_steps(P.d, tile);
    if (assign.out) {
        if (tile == 32) {
            switch (steps) {
                case 1: return launch_waves<32, 1, 2>(NOMAD_ARGS);
                case 2: return launch_waves<32, 2, 2>(NOMAD_ARGS);
                case 4: return launch_waves<32, 4, 2>(NOMAD_ARGS);
                case 6: return launch_waves<32, 6, 2>(NOMAD_ARGS);
                case 8: return launch_waves<32, 8, 2>(NOMAD_ARGS);
                case 12: return launch_waves<32, 12, 2>(NOMAD_ARGS);
                default: return launch_waves<32, 16, 2>(NOMAD_ARGS);
            }
        }
        switch (steps) {
            case 12: return launch_waves<16, 12, 2>(NOMAD_ARGS);
            case 16: return launch_waves<16, 16, 2>(NOMAD_ARGS);
            default: return launch_waves<16, 24, 2>(NOMAD_ARGS);
        }
    }
    if (list_len <= kShortList) {
        if (tile == 32) {
            switch (steps) {
                case 1: return launch_waves<32, 1, 16>(NOMAD_ARGS);
                case 2: return launch_waves<32, 2, 16>(NOMAD_ARGS);
                case 4: return launch_waves<32, 4, 16>(NOMAD_ARGS);
                case 6: return launch_waves<32, 6, 16>(NOMAD_ARGS);
                case 8: return launch_waves<32, 8, 16>(NOMAD_ARGS);
                case 12: return launch_waves<32, 12, 16>(NOMAD_ARGS);
                default: return launch_waves<32, 16, 16>(NOMAD_ARGS);
            }
        }
        switch (steps) {
            case 12: return launch_waves<16, 12, 12>(NOMAD_ARGS);
            case 16: return launch_waves<16, 16, 12>(NOMAD_ARGS);
            default: return launch_waves<16, 24, 12>(NOMAD_ARGS);
        }
    }
    if (tile == 32) {
        switch (steps) {
            case 1: return launch_waves<32, 1, 34>(NOMAD_ARGS);
            case 2: return launch_waves<32, 2, 34>(NOMAD_ARGS);
            case 4: return launch_waves<32, 4, 34>(NOMAD_ARGS);
            case 6: return launch_waves<32, 6, 34>(NOMAD_ARGS);
            default: return launch_waves<32, 8, 34>(NOMAD_ARGS);
        }
    }
    switch (steps) {
        case 6: return launch_waves<16, 6, 20>(NOMAD_ARGS);
        case 8: return launch_waves<16, 8, 20>(NOMAD_ARGS);
        case 12: return launch_waves<16, 12, 20>(NOMAD_ARGS);
        case 16: return launch_waves<16, 16, 20>(NOMAD_ARGS);
        default: return launch_waves<16, 24, 20>(NOMAD_ARGS);
    }
}
