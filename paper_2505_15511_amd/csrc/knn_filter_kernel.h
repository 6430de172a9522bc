// The nearest-neighbour filter for gfx950: what it works on, the kernel, the rules for its shapes.  (knn_kernels.h has the other
// stages and the picture as a whole.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "filter_scale.h"
#include "kmeans_plan.h"

namespace nomad_knn {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int kMaxK = 32;          // neighbours per point
constexpr int kPad = 8;            // extra candidates the filter keeps

// Rows of up to 256 columns are multiplied in 32x32x16 tiles: a wavefront keeps 32 queries in registers (half a kilobyte
// per 16 columns, both parts) and every candidate fragment read from LDS serves 32 of them.  Wider rows, and long lists from
// 128 columns on, leave room for 16 queries per wavefront: 16x16x32 tiles.
constexpr int kShortList = 24;     // K' up to which the short lists are used
__host__ __device__ constexpr int knn_tile(int d, int list_len) { return d <= (list_len <= kShortList ? 256 : 128) ? 32 : 16; }
// matrix steps (of 512 / tile columns) the kernels are compiled for
__host__ __device__ constexpr int knn_steps(int d, int tile) {
    return tile == 32 ? (d <= 16 ? 1 : d <= 32 ? 2 : d <= 64 ? 4 : d <= 96 ? 6 : d <= 128 ? 8 : d <= 192 ? 12 : 16)
                      : (d <= 192 ? 6 : d <= 256 ? 8 : d <= 384 ? 12 : d <= 512 ? 16 : 24);
}
__host__ __device__ constexpr size_t knn_tile_units(int steps) { return (size_t)steps * 2 * 64; }   // 16-byte units of a packed tile

struct KnnBlock { int32_t cluster; int32_t q0; };   // one workgroup's share: tiles (or rows) q0 .. of group `cluster`

// Rows laid out for the matrix cores (k_knn_pack): every group's rows in tiles of knn_tile(d), the last one padded.
struct KnnPacked {
    const uint4* data;           // [tiles][steps][hi, lo][64 lanes] 16 bytes: lane l of a step holds columns 8 (l / tile) .. + 7 of row l % tile
    const float* norm;           // [tiles][tile] |x'|^2 / 2 (float32, of the centred row) in units of both sides' scales, +inf in the padding
    const uint32_t* tstart;      // [groups + 1] first tile of every group
    const uint32_t* max_bits;    // [groups] largest |x'|^2 of the group's rows: the scale of the group
};

// Queries and candidates, both cut into the same groups (group g: queries qmembers[qstart[g] .. qstart[g+1]), candidates
// cmembers[cstart[g] .. cstart[g+1])).  Nearest neighbours inside clusters: both are the data set grouped by cluster.
// K-Means assignment: one group, the queries are the points, the candidates the centroids.  Neighbourhoods of a sample
// of query points among all points: one group, the queries a gathered copy of the sampled rows.
struct KnnSets {
    const float* XQ;             // query rows
    const float* XC;             // candidate rows
    const int32_t* qmembers;     // query row of every position, or nullptr = the position itself
    const int32_t* cmembers;     // candidate row of every position, or nullptr = the position itself
    const uint32_t* qstart;      // [groups + 1]
    const uint32_t* cstart;      // [groups + 1]
    KnnPacked Q, C;              // both sides packed
    const float* centre;         // [groups][d] what both sides are centred on
    const int32_t* group_of_q;   // group of every query row, or nullptr = group 0
    int64_t n_q, n_c;            // rows of XQ, XC
    int32_t d;
    int32_t same_set;            // 1: queries and candidates are the same rows: a row is not its own neighbour
    int32_t chunk;               // columns that the filter sums at a time (knn_chunk_columns): its error bound depends on it
    const int32_t* self_row;     // or, per query row, the candidate row that is the query itself (nullptr: see same_set)
    int32_t ordered;             // 1: the rows of a group lie cell by cell (k_knn_place): near rows are near in the list
    // The groups are slices of one set, each with the same queries in the same order, and the answer is the nearest of all slices: what the others
    // have found bounds what a slice has to find (nullptr: the groups have nothing to do with each other).
    void* shared;                // [slices][queries][lanes of a query][4] squared distances that share_rank, 2, 3, 4 share_rank candidates of the lane are within; large at first
    const float* q_norm;         // [n_q] |x'|^2 of the queries
    int32_t slices, share_rank;
    // One neighbour wanted: the large products alone (k_knn_filter), and where the queries are counted that these leave open, or would (nullptr:
    // nowhere); q_norm is there then
    int32_t alone;
    uint32_t* open_count;
};

__device__ __forceinline__ int32_t knn_row(const int32_t* members, uint32_t pos) { return members ? members[pos] : (int32_t)pos; }

// ---------------------------------------------------------------- stage 1: the filter on the matrix cores
template <int TILE> struct MatrixTile;
template <> struct MatrixTile<32> {
    typedef float Acc __attribute__((ext_vector_type(16)));
    static __device__ __forceinline__ Acc mul(half8 a, half8 b, Acc c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};
template <> struct MatrixTile<16> {
    typedef float Acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Acc mul(half8 a, half8 b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};

// Tiles staged together, and stages in LDS.  Lists of several neighbours: two stages of up to 24 steps; a wavefront that inserts
// or cannot sift falls behind, and the others wait for it once a stage: three tiles of 128 columns against two (three buffers,
// the same LDS) are 1.5 % of a filter over large clusters and 1 % of one over slices of the whole set; two workgroups of four
// wavefronts per unit, which wait for each other less but stage every tile twice, are 10 and 5 % slower.  Otherwise loads into
// LDS are issued two stages ahead of their use (one at the widest rows, whose stages are 48 KB), which is what hides the
// memory's latency behind 3,000 cycles of matrix instructions per stage.  Twelve and sixteen wavefronts leave LDS for two stages of 16 and 8 steps.
// Steps of the large products that are summed by themselves (0: all of them in one sum): 64 columns.  The bound on a sum's
// rounding grows with its length, and with the bound the number of candidates whose order the keys leave open and whose rows
// k_knn_refine has to read, and of queries left to the exact path.  1,000,000 x 128 in clusters of 4,000, sums of all columns /
// 64 / 32: filter 5.33 / 5.42 / 5.4 ms, refinement 0.91 / 0.74 / 0.65, exact path 0.09 / 0.05 / 0.04; but over slices of the
// whole set the additions cost more than they save (7.9 / 7.9 / 8.2 ms a call).  One neighbour wanted: the lists hold two and the
// bound decides few (partition of 1,000,000 x 128: no gain).  Not where registers would spill: the widest rows with one neighbour
// (95 -> 123 us of filter for 8 us of exact path), long lists and more than 192 columns in 32-row tiles.
__host__ __device__ constexpr int knn_chunk_steps(int tile, int steps, int L) {
    const int chunk = 64 * tile / 512;
    return steps <= chunk ? 0 : (tile == 16 ? L > 2 || steps <= 16 : L == 16 && steps <= 12) ? chunk : 0;
}
constexpr int kMaxStageTiles = 16;   // packed arrays are this many tiles longer than what they hold
__host__ __device__ constexpr int knn_stage_tiles(int tile, int steps, int L, int waves, int parts = 2) {
    const int target = tile == 16 ? steps : parts == 1 ? 16 : waves > 12 ? 8 : waves > 8 ? 16 : (L > 2 && waves == 8) ? 24 : 8;
    return steps >= target ? 1 : target / steps < kMaxStageTiles ? target / steps : kMaxStageTiles;
}
__host__ __device__ constexpr int knn_buffers(int tile, int steps, int L, int waves) {
    return (tile == 16 && steps > 16) || (L > 2 && waves >= 8 && knn_stage_tiles(tile, steps, L, waves) > 1) ? 2 : 3;
}
__host__ __device__ constexpr int knn_fifo(int tile) { return tile == 32 ? 12 : 8; }   // hits a lane sets aside before they go into its list
// (parts: 2, or 1 where only the high halves are staged)
__host__ __device__ constexpr size_t knn_stage_bytes(int tile, int steps, int L, int waves, int parts) {
    return (size_t)knn_stage_tiles(tile, steps, L, waves, parts) * (knn_tile_units(steps) / 2 * parts * 16 + (size_t)tile * 4);
}
__host__ __device__ constexpr size_t knn_filter_lds_bytes(int tile, int steps, int L, int waves, int parts) {
    return knn_buffers(tile, steps, L, waves) * knn_stage_bytes(tile, steps, L, waves, parts) + (L > 2 ? (size_t)waves * knn_fifo(tile) * 64 * 8 : 0);
}
// whether a filter that sifts has the other way of multiplying a tile too (see below): not where registers are short
__host__ __device__ constexpr bool knn_both_ways(int tile, int steps, int waves) { return waves <= 8 && !(tile == 16 && steps > 16); }
__host__ __device__ constexpr int knn_waves_per_simd(int tile, int steps, int L, int waves) {
    return waves > 8 ? waves / 4 : waves != 8 ? 1 : tile == 32 && L == 2 && steps <= 8 ? 4 : 2;
}

// 16 (4) bytes per lane from global memory straight into LDS: lane l's go to byte offset `to` + 16 l (4 l).  Not known to the
// compiler as a load: the caller waits with wait_loads, and reads what has arrived only behind a barrier.
__device__ __forceinline__ void load_to_lds16(uint32_t to, const void* base, uint32_t byte_offset) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(byte_offset), "s"(base) : "m0", "memory");
}
__device__ __forceinline__ void load_to_lds4(uint32_t to, const void* base, uint32_t byte_offset) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(to), "v"(byte_offset), "s"(base) : "m0", "memory");
}
template <int LEFT>   // until at most LEFT of this wavefront's loads are outstanding
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LEFT) : "memory"); }

// One workgroup = WAVES tiles of queries of one group, one tile per wavefront, looping over the group's candidate tiles.
// A = the candidates, B = the negated queries, C = |c|^2 / 2: the matrix instructions leave half of the key, |c|^2 - 2 q.c,
// in units of the scales.  Lane l supplies row l % TILE and columns 8 (l / TILE) .. + 7 of a step; D: lane l holds query
// l % TILE and the candidates 8 (v / 4) + 4 (l / TILE) + v % 4 in element v.  The queries' fragments stay in registers, the
// candidates' tiles come packed and are loaded straight into LDS, a stage of tiles at a time.
//
// float16 matrix instructions run at 16 times the rate of the float32 ones (2.5 PFLOP/s against 157 TFLOP/s), so three
// products cost a fifth of one in float32; unlike those they also leave the vector pipe to the selection.
//
// Sifting: the products hi lo + lo hi, two thirds of the matrix work, are at most `slack` in size (Cauchy-Schwarz, from the
// query's own parts and the largest candidate).  The large product comes first and the others follow only where some lane's smallest
// key comes within slack of its threshold.  The keys are the same bits, and what is passed over would not have been looked at.
// Where the rows of a group lie cell by cell (P.ordered) the scan begins at the queries' own tiles, whose candidates bring the
// thresholds down, and of the other cells' tiles few are left: 1,000,000 x 128 in clusters of 4,000, 47 % of the tiles end there.
// Multiplying the large product first also needs a third accumulator less, and with it three wavefronts a SIMD fit the registers (four of
// the shortest rows), which is worth as much: filter 4.9 ms, ordered 4.2, with twelve wavefronts a workgroup 3.8.  In random order
// few tiles hold no hit until far into a long group (TILE K' of TILE t candidates' keys after t tiles): there workgroups of eight
// wavefronts multiply all three products side by side up to tile TILE K' / 2, which saves a chain of dependent products a tile.
// 10,000 queries among 1,000,000 x 128 in six slices: 63 % of the tiles end after the large product, the filter takes 5.96 ms instead of 7.6, and 4.5 since
// the slices tell each other their distances (5.1 with one rank a list; 3.1 is what it takes without any hit).
// Workgroups of fewer wavefronts (few queries, one wavefront a SIMD) have nobody to multiply while a chain of dependent products is
// waited for, and a tile with a hit then waits for two chains in turn: they sift from tile 2 TILE K' on.  50 queries, 30 neighbours,
// 300,000 x 400: filter 2.18 ms without sifting and chunks, 2.53 with both, 2.41 with the later start and 2.38 with a chunk's sum
// added while the next one is multiplied.  Rows of more than 512 columns have registers for one way only (both: 32 to 63 spilled, call
// +10 %): sifting where the rows are ordered, side by side otherwise.
//
// Selection: 64 / TILE lanes share a query, each sees its part of every tile's candidates and keeps the L smallest keys,
// with their positions, sorted in registers.  Keys below the lane's threshold are set aside in a small queue in LDS; when a
// lane's queue is nearly full every lane of the wavefront inserts what it has, one entry per pass (a sorted slot becomes
// the median of its left neighbour, the new key and itself).  Inserting at once would spend a pass of the whole wavefront
// on nearly every tile; the queue fills its passes.  Keys are looked at in fours: one comparison and a branch where no lane
// of the wavefront has a hit.  The threshold is the smaller of the lane's last key and the largest of
// the lanes' H-th keys (H 64 / TILE >= K': what lies above that is not among the K' smallest).
// Slices of one set (P.shared) tell each other how far their lists reach: every lane's r-th, 2 r-th, 3 r-th and 4 r-th keys, with r so that the 2 r-th of all
// lists together are K' candidates.  The least distance within which those that have told theirs hold K' of them (up to 8 slices; beyond, the least of the four ranks'
// largest that do) is not below the K'-th nearest of the set, and a slice need not look at what lies above it.  As distances, for the slices' centres
// differ; raised by twice the filter's error bound where they are written and where they are read, and by more than the conversion's roundings, so that what is
// turned away on their account is farther than the K'-th nearest for certain, and `tau` speaks of the rest only.  Every wavefront writes its
// queries' and reads the others' whenever it has seen an eighth more (some forty times; what others have not written yet bounds nothing, nobody waits).
// In a launch of several rounds the later slices begin with the bound of the earlier ones: 300,000 x 128, 17,000 queries in 15 slices 5.35 -> 4.80 ms against a bound
// that needs all lists, 150,000 x 20 among themselves in 3 slices 9.9 -> 9.1.
// At the end the lists are merged by counting, smallest key first; tau = min(K'-th key of the union, the lists' last keys): every candidate
// that is not passed on has key >= tau, or another slice's distances rule it out.
//
// L == 2: one neighbour wanted.  Every key goes straight into the lane's best two; at the end a query whose smallest key
// lies below the second by more than twice the filter's error bound has its answer (out); the others are put on the `todo`
// list (query position in todo, its 2 * 64 / TILE candidates in cand, tau) for k_assign_refine.
//
// Large products alone: the nearest centroid is usually nearer than the second by more than 2 slack, and then hi hi decides: a third of the
// products, and half of what is read of the queries.  A step of Lloyd's iterations does without the others where the one before has
// left (or, with all three products, would have left) few of the queries open (products_alone); the first one does not.  What is open goes to
// k_assign_refine as ever, with slack in the margin and in tau.  1,000,000 x 128 and 256 centroids: 227 -> 132 us a step, a call of ten 4.64 -> 3.76 ms (before keys were numbered: 196 and 104).
// Or, with `open`, a word of bits a tile of queries says which those are, and what goes with them lies at their positions (a list's one counter was what
// the step waited for: a step of a million points with one in every second wavefront, 150 us for 132).
struct KnnAssign { int32_t* out; int32_t* todo; uint32_t* n_todo; uint32_t* open; };

// What an instance does beside the common part; each is compiled for itself, since scalar registers and the code before the loop count in short groups
// (6,582 x 84 in 25 clusters with the slices' exchange compiled in: a call 169 -> 178 us)
enum FilterWay : int {
    kWaySift,      // several neighbours: sifts
    kWayBeside,    // several neighbours: all three products side by side
    kWayShare,     // several neighbours: sifts, and the groups are slices that share their distances
    kWayAlone      // one neighbour: the large products alone
};
// whether an instance for slices exists: not where registers are short
__host__ __device__ constexpr bool knn_shares(int tile, int steps, int L) { return L > 2 && knn_both_ways(tile, steps, 8) && !(tile == 32 && steps > 12); }

template <int TILE, int KS, int L, int WAVES, int WAY = kWaySift>
__global__ void __launch_bounds__(64 * WAVES, knn_waves_per_simd(TILE, KS, L, WAVES)) k_knn_filter(const KnnSets P, const KnnBlock* __restrict__ blocks, int32_t list_len,
                                                                               int32_t* __restrict__ cand, float* __restrict__ key_out, float* __restrict__ tau_out,
                                                                               const KnnAssign assign) {
    using Mat = MatrixTile<TILE>;
    using Acc = typename Mat::Acc;
    constexpr int kShare = 64 / TILE;                 // lanes per query
    constexpr int kKeys = TILE * TILE / 64;           // keys per lane and tile
    constexpr bool kAlone = WAY == kWayAlone;          // large products alone
    constexpr int kParts = kAlone ? 1 : 2;
    constexpr int kUnits = KS * 2 * 64, kStaged = KS * kParts * 64;   // 16-byte units of a tile, of what is staged of it
    constexpr int kChunk = knn_chunk_steps(TILE, KS, L);
    constexpr int kStage = knn_stage_tiles(TILE, KS, L, WAVES, kParts), kBuffers = knn_buffers(TILE, KS, L, WAVES);
    constexpr int kStageBytes = (int)knn_stage_bytes(TILE, KS, L, WAVES, kParts), kDataBytes = kStage * kStaged * 16;
    constexpr int kCopies = (kStage * KS * kParts + WAVES - 1) / WAVES;              // 1 KB loads of a wavefront per stage
    constexpr int kNormCopies = (kStage * TILE + 63) / 64;                      // (every wavefront loads all the norms: they are few)
    constexpr int kLoads = kCopies + kNormCopies;
    constexpr int F = knn_fifo(TILE);
    constexpr int H = TILE == 32 ? (L == 16 ? 12 : 20) : (L == 12 ? 6 : 10);   // H * kShare >= the largest K' of the class
    extern __shared__ uint4 lds[];                    // [kBuffers] stages: tiles, then their norms; then the queues
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), part = lane / TILE;
    const KnnBlock blk = blocks[blockIdx.x];
    const int32_t grp = blk.cluster;
    if (grp < 0) return;                                      // no work: fills a list up
    const uint32_t c0 = P.cstart[grp], ct0 = P.C.tstart[grp];
    // a group whose keys are not all finite (knn_filter_usable) passes nothing on: its queries are the exact path's
    const int32_t n_tiles = knn_filter_usable(P.Q.max_bits[grp], P.C.max_bits[grp]) ? (int32_t)(P.C.tstart[grp + 1] - ct0) : 0;
    const uint32_t q0g = P.qstart[grp];
    const int32_t n_qg = (int32_t)(P.qstart[grp + 1] - q0g);
    const uint32_t qt = P.Q.tstart[grp] + (uint32_t)(blk.q0 + wave);
    const bool live = qt < P.Q.tstart[grp + 1];               // wave-uniform
    const int32_t qpos = (blk.q0 + wave) * TILE + (lane & (TILE - 1));
    const int32_t qpt = live && qpos < n_qg ? knn_row(P.qmembers, q0g + (uint32_t)qpos) : -1;
    // position of the candidate that is the query itself, if any
    const int32_t self = qpt < 0 ? -1 : P.self_row ? P.self_row[qpt] - (int32_t)c0 : P.same_set ? qpos : -1;
    half8 bh[KS], bl[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        uint4 h = make_uint4(0u, 0u, 0u, 0u), l = h;
        if (live) {
            const uint4* src = P.Q.data + ((size_t)qt * KS + s) * 128 + lane;
            h = src[0];
            if (!kAlone) l = src[64];
        }
        constexpr uint32_t kSign = 0x80008000u;
        h.x ^= kSign; h.y ^= kSign; h.z ^= kSign; h.w ^= kSign;
        l.x ^= kSign; l.y ^= kSign; l.z ^= kSign; l.w ^= kSign;
        bh[s] = *(const half8*)&h;
        bl[s] = *(const half8*)&l;
    }
    // half keys in units of both scales
    const int unit_exp = knn_scale_exponent(P.Q.max_bits[grp]) + knn_scale_exponent(P.C.max_bits[grp]);
    const float key_unit = ldexpf(2.f, -unit_exp);
    float lk[L];
    int32_t lp[L];
#pragma unroll
    for (int x = 0; x < L; ++x) { lk[x] = __builtin_inff(); lp[x] = -1; }
    float thr = qpt >= 0 ? __builtin_inff() : -__builtin_inff();   // lanes without a query take nothing
    float others_thr = __builtin_inff();                           // what the other slices have made of it

    const char* csrc = (const char*)(P.C.data + (size_t)ct0 * kUnits);
    const char* nsrc = (const char*)(P.C.norm + (size_t)ct0 * TILE);
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)(char*)lds;
    // the lanes' queues [WAVES][F][keys, positions][64]: an entry is kEntry bytes after the one before; `at` is where the lane's
    // next one goes, and a lane has more than x of them when at lies above queue0 + x kEntry + 255
    constexpr uint32_t kEntry = 512;
    const uint32_t queue0 = lds0 + (uint32_t)(kBuffers * kStageBytes) + (uint32_t)wave * (F * kEntry);
    uint32_t at = queue0 + 4u * (uint32_t)lane;
    const auto holds_more_than = [&](int x) { return at > queue0 + (uint32_t)x * kEntry + 255u; };
    const int32_t n_stages = (n_tiles + kStage - 1) / kStage;
    // first stage: the one the queries themselves are in, where what is near them is there too
    const int32_t stage0 = P.ordered ? min(blk.q0 / kStage, max(n_stages - 1, 0)) : 0;
    const auto first_tile = [&](int32_t x) {   // of the x-th stage, all of them in turn from stage0 on
        x += stage0;
        return (x >= n_stages ? x - n_stages : x) * kStage;
    };
    // the x-th stage (the last one again where that is past the end), into buffer buf.  The group's last stage may
    // take tiles beyond the group's along; the arrays are long enough for that, and nobody looks at them.
    auto fetch = [&](int32_t x, int buf) {
        const int32_t t = first_tile(min(x, n_stages - 1));
        const char* from = csrc + (size_t)t * kUnits * 16;
        const uint32_t to = lds0 + (uint32_t)(buf * kStageBytes);
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            const uint32_t at = (uint32_t)min(wave + u * WAVES, kStage * KS * kParts - 1) * 1024u;
            load_to_lds16(to + at, from, at * (uint32_t)(2 / kParts) + (uint32_t)lane * 16u);
        }
        const char* nfrom = nsrc + (size_t)t * TILE * 4;
#pragma unroll
        for (int u = 0; u < kNormCopies; ++u)
            if (kStage * TILE % 64 == 0 || u * 64 + lane < kStage * TILE) load_to_lds4(to + kDataBytes + u * 256, nfrom, (uint32_t)(u * 64 + lane) * 4u);
    };
    // one entry of every lane's queue into its list, from the last slot down, in place (the empty assembly keeps the slots in
    // their registers: left to itself the compiler copies the whole list every pass)
    auto insert = [&](float xk, int32_t xp) {
        bool here = xk < lk[L - 1];
#pragma unroll
        for (int x = L - 1; x >= 1; --x) {
            const bool left = xk < lk[x - 1];
            const int32_t moved = left ? lp[x - 1] : xp;
            lp[x] = here ? moved : lp[x];
            lk[x] = __builtin_amdgcn_fmed3f(lk[x - 1], xk, lk[x]);
            asm volatile("" : "+v"(lk[x]), "+v"(lp[x]));
            here = left;
        }
        lp[0] = here ? xp : lp[0];
        lk[0] = here ? xk : lk[0];
        asm volatile("" : "+v"(lk[0]), "+v"(lp[0]));
    };
    // passes until no lane's queue holds more than `level` entries, newest first; the next pass's entries are read a pass ahead
    // (a lane without one reads the place of its first)
    auto drain = [&](int level) {
        typedef __attribute__((address_space(3))) const float Lds;
        bool has = holds_more_than(0), more = __any(holds_more_than(level));
        uint32_t from = has ? at - kEntry : at;
        float k = *(Lds*)from, p = *(Lds*)(from + 256u);
        while (more) {
            const float xk = has && __float_as_int(p) != self ? k : __builtin_inff();
            const int32_t xp = __float_as_int(p);
            at = from;
            more = __any(holds_more_than(level));
            has = holds_more_than(0);
            from = has ? at - kEntry : at;
            k = *(Lds*)from;
            p = *(Lds*)(from + 256u);
            insert(xk, xp);
        }
        float most = lk[H < L ? H - 1 : 0];
#pragma unroll
        for (int w = TILE; w < 64; w <<= 1) most = fmaxf(most, __shfl_xor(most, w, 64));
        if (qpt >= 0) thr = fminf(fminf(lk[L - 1], most), others_thr);
    };
    // ranks published of every lane's list: r, 2 r, 3 r, 4 r, r = P.share_rank
    constexpr int kBisect = 8, kFine = 8;
    const auto share = [&]() {
        const float eps2 = 2.01f * (float)knn_filter_eps(P.d, fmax((double)__uint_as_float(P.Q.max_bits[grp]), (double)__uint_as_float(P.C.max_bits[grp])), kChunk * 512 / TILE);
        const int32_t row = max(qpt, 0), m = n_qg * kShare, mine = min(qpos, n_qg - 1) * kShare + part;   // (lanes without a query go along)
        const float qn = P.q_norm[row], least = fmaf(qn, 1e-4f, eps2);
        float own[4];
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const int at_rank = (y + 1) * P.share_rank - 1;
            float v = lk[0];
#pragma unroll
            for (int x = 1; x < L; ++x) v = x == at_rank ? lk[x] : v;
            own[y] = fminf(fmaf(v, key_unit, qn) + least, 3e38f);
        }
        unsigned long long* const lists = (unsigned long long*)P.shared;
        const auto both = [](float a, float b) { return (unsigned long long)__float_as_uint(b) << 32 | __float_as_uint(a); };
        if (qpt >= 0) {
            unsigned long long* const to = lists + ((size_t)grp * m + mine) * 2;
            __hip_atomic_store(to, both(own[0], own[1]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(to + 1, both(own[2], own[3]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // of each of the four ranks, how many lists have told theirs, and the largest of these distances: what `far` is taken from
        float near = own[0], most[4] = {0.f, 0.f, 0.f, 0.f}, o[kFine][4];
        int told[4] = {0, 0, 0, 0};
        for (int32_t h0 = 0; h0 < P.slices; h0 += kFine) {
            unsigned long long lo[kFine], hi[kFine];
#pragma unroll
            for (int u = 0; u < kFine; ++u) {
                const unsigned long long* const from = lists + ((size_t)min(h0 + u, P.slices - 1) * m + mine) * 2;
                lo[u] = __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                hi[u] = __hip_atomic_load(from + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int u = 0; u < kFine; ++u) {
                o[u][0] = __uint_as_float((uint32_t)lo[u]); o[u][1] = __uint_as_float((uint32_t)(lo[u] >> 32));
                o[u][2] = __uint_as_float((uint32_t)hi[u]); o[u][3] = __uint_as_float((uint32_t)(hi[u] >> 32));
                if (h0 + u >= P.slices) o[u][0] = o[u][1] = o[u][2] = o[u][3] = 3e38f;
                near = fminf(near, o[u][0]);
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const bool has = o[u][y] < 1e30f;
                    told[y] += has ? 1 : 0;
                    most[y] = fmaxf(most[y], has ? o[u][y] : 0.f);
                }
            }
        }
        float far = __builtin_inff();
#pragma unroll
        for (int y = 0; y < 4; ++y) {
#pragma unroll
            for (int w = TILE; w < 64; w <<= 1) { told[y] += __shfl_xor(told[y], w, 64); most[y] = fmaxf(most[y], __shfl_xor(most[y], w, 64)); }
            if (told[y] * (y + 1) * P.share_rank >= list_len) far = fminf(far, most[y]);
        }
        if (!__any(far < 1e30f)) return;   // too few lists have told theirs
#pragma unroll
        for (int w = TILE; w < 64; w <<= 1) near = fminf(near, __shfl_xor(near, w, 64));
        if (P.slices <= kFine) {   // the lists are all in registers: the least distance that K' candidates are within, or a little more
            for (int y = 0; y < kBisect; ++y) {
                const float mid = 0.5f * (near + far);
                int within = 0;
#pragma unroll
                for (int u = 0; u < kFine; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) within += o[u][v] <= mid ? 1 : 0;
#pragma unroll
                for (int w = TILE; w < 64; w <<= 1) within += __shfl_xor(within, w, 64);
                if (within * P.share_rank >= list_len) far = mid;
                else near = mid;
            }
        }
        if (qpt >= 0 && far > 1e-30f && far < 1e30f) {   // (elsewhere roundings are not what `least` covers)
            others_thr = fminf(others_thr, ldexpf(fmaf(far, 1.000001f, least - qn), unit_exp - 1));
            thr = fminf(thr, others_thr);
        }
    };
    // key and position into the queues of the lanes whose key lies below their threshold: a mask and no branch.  (A branch a key,
    // two jumps on most keys of short groups, and reading a queue's entry only when its pass begins: calls with 1,000,000 x 128 in
    // 256 clusters took 6.70 ms, now 6.22.)
    auto push = [&](float key, int32_t pos) {
        unsigned long long all;
        asm volatile("v_cmp_lt_f32_e32 vcc, %[key], %[thr]\n\t"
                     "s_and_saveexec_b64 %[all], vcc\n\t"
                     "ds_write2st64_b32 %[at], %[key], %[pos] offset0:0 offset1:1\n\t"
                     "v_add_u32_e32 %[at], %[entry], %[at]\n\t"
                     "s_mov_b64 exec, %[all]"
                     : [at] "+v"(at), [all] "=&s"(all)
                     : [key] "v"(key), [thr] "v"(thr), [pos] "v"(pos), [entry] "s"(kEntry)
                     : "vcc", "scc", "memory");
    };
    constexpr bool kShares = WAY == kWayShare;
    constexpr bool kSift = L > 2 && WAY != kWayBeside, kTogether = knn_both_ways(TILE, KS, WAVES) || WAY == kWayBeside;
    // step s of the large product: big = the norms and the chunks before, chunk = the present one
    const auto large = [&](Acc& big, Acc& chunk, half8 a, int s) {
        if (kChunk == 0 || s < kChunk) { big = Mat::mul(a, bh[s], big); return; }
        if (s % (kChunk ? kChunk : 1) == 0) {
            const Acc before = chunk;
            chunk = Acc{};
            if (WAVES >= 8 && s > kChunk) big += before;
            chunk = Mat::mul(a, bh[s], chunk);
            if (WAVES < 8 && s > kChunk) {
                __builtin_amdgcn_sched_barrier(0);     // the chunk before is added while this one is multiplied
                big += before;
            }
        } else {
            chunk = Mat::mul(a, bh[s], chunk);
        }
        if (s == KS - 1) big += chunk;
    };
    // One neighbour, in 32-row tiles: the element v of the accumulator goes into the last four bits of the key, so that the two smallest of a tile's sixteen take three instructions a key instead of
    // eight; those keys differ from their own by less than 2^-19 of them, which the margin and tau carry.  A group's last tile, if padded, is done key by key
    // (infinity with a number in it is none; keys of a full tile are finite, knn_filter_usable).  Points that this leaves open besides, simulated on mixtures and noise of 8 to 768 columns: with all
    // three products up to 70 of a million (750 to 1,800 are), with the large ones alone, whose margin is a hundred times as wide, up to 30 (33,000 to 70,000 are).  Large products alone, 1,000,000 x 128 on 256 centroids: 132 -> 104 us a step, with all three products 222 -> 196.
    constexpr bool kNumbered = L == 2 && TILE == 32;
    // positions there: 16 times the tile and the element, which is candidate 8 (v / 4) + 4 part + v % 4 of the tile
    const auto place_of = [&](int32_t p) { return p < 0 || !kNumbered ? p : (p >> 4) * TILE + 8 * (p >> 2 & 3) + 4 * part + (p & 3); };
    const int32_t n_cands = (int32_t)(P.cstart[grp + 1] - c0);
    const int32_t sift_from = !kSift ? n_tiles : !kTogether || P.ordered ? 0 : (WAVES == 8 ? list_len * TILE / 2 : list_len * TILE * 2) / (kShares ? P.slices : 1);
    float slack = 0.f;             // >= |hi lo + lo hi| of this query with any candidate, as summed below
    // |hi| <= |c| (1 + 2^-11), |lo| <= 2^-11 |c|, below float16's normal numbers 2^-25 an element; one part in a hundred for
    // the roundings of the sums (2 768 terms of 2^-23 at most) and of max_bits
    const auto longest_candidate = [&]() { return ldexpf(sqrtf(__uint_as_float(P.C.max_bits[grp])), knn_scale_exponent(P.C.max_bits[grp])); };
    const auto least_part = [&]() { return sqrtf((float)P.d) * 0x1p-25f; };
    if (kSift && sift_from < n_tiles) {
        float h2 = 0.f, l2 = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                h2 = fmaf((float)bh[s][v], (float)bh[s][v], h2);
                l2 = fmaf((float)bl[s][v], (float)bl[s][v], l2);
            }
#pragma unroll
        for (int w = TILE; w < 64; w <<= 1) { h2 += __shfl_xor(h2, w, 64); l2 += __shfl_xor(l2, w, 64); }
        const float longest = longest_candidate(), least = least_part();
        slack = 1.01f * (sqrtf(l2) * (1.001f * longest + least) + sqrtf(h2) * (0x1p-11f * longest + least));
    }
    // tile number i of the stage in buffer `buf`, tile t of the group, `before` tiles after the first
    auto consume = [&](int buf, int i, int32_t t, int32_t before) {
        const char* stage = (const char*)lds + buf * kStageBytes;
        const float* nn = (const float*)(stage + kDataBytes) + i * TILE + 4 * part;
        const uint4* frag = (const uint4*)stage + i * kStaged + lane;
        Acc big, small;
#pragma unroll
        for (int g = 0; g < kKeys / 4; ++g) {
            const float4 n4 = *(const float4*)(nn + 8 * g);
            big[4 * g] = n4.x; big[4 * g + 1] = n4.y; big[4 * g + 2] = n4.z; big[4 * g + 3] = n4.w;
        }
        if (kSift && (!kTogether || before >= sift_from)) {
            constexpr int kAhead = KS < 4 ? KS : 4;    // steps whose fragments are on their way
            half8 a[kAhead];
#pragma unroll
            for (int s = 0; s < kAhead; ++s) a[s] = *(const half8*)&frag[s * 128];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                __builtin_amdgcn_sched_barrier(0);
                large(big, small, a[s % kAhead], s);
                __builtin_amdgcn_sched_barrier(0);
                if (s + kAhead < KS) a[s % kAhead] = *(const half8*)&frag[(s + kAhead) * 128];
            }
            float low = big[0];
#pragma unroll
            for (int v = 1; v < kKeys; ++v) low = fminf(low, big[v]);
            if (!__any(low <= thr + slack)) return;    // (a key below thr, big + small rounded, has big <= thr + |small|)
#pragma unroll
            for (int v = 0; v < kKeys; ++v) small[v] = 0.f;
            half8 ah = *(const half8*)&frag[0], al = *(const half8*)&frag[64];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                half8 nh = ah, nl = al;
                if (s + 1 < KS) { nh = *(const half8*)&frag[(s + 1) * 128]; nl = *(const half8*)&frag[(s + 1) * 128 + 64]; }
                __builtin_amdgcn_sched_barrier(0);
                small = Mat::mul(ah, bl[s], small);
                small = Mat::mul(al, bh[s], small);
                __builtin_amdgcn_sched_barrier(0);
                ah = nh;
                al = nl;
            }
        } else if (kAlone) {
            constexpr int kAhead = KS < 4 ? KS : 4;
            half8 a[kAhead];
#pragma unroll
            for (int s = 0; s < kAhead; ++s) a[s] = *(const half8*)&frag[s * 64];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                __builtin_amdgcn_sched_barrier(0);
                large(big, small, a[s % kAhead], s);
                __builtin_amdgcn_sched_barrier(0);
                if (s + kAhead < KS) a[s % kAhead] = *(const half8*)&frag[(s + kAhead) * 64];
            }
        } else {
            Acc chunk;
#pragma unroll
            for (int v = 0; v < kKeys; ++v) small[v] = 0.f;
            half8 ah = *(const half8*)&frag[0], al = *(const half8*)&frag[64];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                half8 nh = ah, nl = al;
                if (s + 1 < KS) { nh = *(const half8*)&frag[(s + 1) * 128]; nl = *(const half8*)&frag[(s + 1) * 128 + 64]; }
                __builtin_amdgcn_sched_barrier(0);     // the next step's fragments are on their way while this step is multiplied
                small = Mat::mul(ah, bl[s], small);
                large(big, chunk, ah, s);
                small = Mat::mul(al, bh[s], small);
                __builtin_amdgcn_sched_barrier(0);
                ah = nh;
                al = nl;
            }
            if (L == 2) big += small;
        }
        if (kNumbered && (t + 1) * TILE <= n_cands) {
            float k0 = __builtin_inff(), k1 = k0;   // the two smallest of the tile's keys, numbered
#pragma unroll
            for (int v = 0; v < kKeys; ++v) {
                const float key = __uint_as_float((__float_as_uint(big[v]) & 0xFFFFFFF0u) | (uint32_t)v);
                k1 = __builtin_amdgcn_fmed3f(k0, key, k1);
                asm("v_min_f32_e32 %0, %1, %2" : "=v"(k0) : "v"(key), "v"(k0));   // (fminf would make sure first that neither is a signalling NaN)
            }
            const int32_t p0 = t << 4 | (int32_t)(__float_as_uint(k0) & 15u), p1 = t << 4 | (int32_t)(__float_as_uint(k1) & 15u);
            const bool lt0 = k0 < lk[0], lt1 = k0 < lk[L - 1];
            lp[L - 1] = lt0 ? lp[0] : (lt1 ? p0 : lp[L - 1]);
            lk[L - 1] = __builtin_amdgcn_fmed3f(lk[0], k0, lk[L - 1]);
            lp[0] = lt0 ? p0 : lp[0];
            lk[0] = lt0 ? k0 : lk[0];
            const bool second = k1 < lk[L - 1];     // (not below the first: k0 is not)
            lp[L - 1] = second ? p1 : lp[L - 1];
            lk[L - 1] = second ? k1 : lk[L - 1];
            return;
        }
#pragma unroll
        for (int g = 0; g < kKeys / 4; ++g) {
            float key[4];
            const int32_t pos0 = t * TILE + 8 * g + 4 * part;
#pragma unroll
            for (int v = 0; v < 4; ++v) key[v] = L == 2 ? big[4 * g + v] : big[4 * g + v] + small[4 * g + v];
            if (L == 2) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int32_t at_v = kNumbered ? t << 4 | (4 * g + v) : pos0 + v;   // (see place_of)
                    const bool lt0 = key[v] < lk[0], lt1 = key[v] < lk[L - 1];
                    lp[L - 1] = lt0 ? lp[0] : (lt1 ? at_v : lp[L - 1]);
                    lk[L - 1] = __builtin_amdgcn_fmed3f(lk[0], key[v], lk[L - 1]);
                    lp[0] = lt0 ? at_v : lp[0];
                    lk[0] = lt0 ? key[v] : lk[0];
                }
            } else if (__any(fminf(fminf(key[0], key[1]), fminf(key[2], key[3])) < thr)) {
#pragma unroll
                for (int v = 0; v < 4; ++v) push(key[v], pos0 + v);
                if (__any(holds_more_than(F - 4))) drain(F - 8);
            }
        }
        if (L > 2 && __any(holds_more_than(4))) drain(4);
    };

    // the queries' fragments are here before the loop begins: a wait for them inside it would be a wait for the stage's loads
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(bh[s]), "+v"(bl[s]));
    if (n_tiles > 0) {
#pragma unroll
        for (int x = 0; x < kBuffers - 1; ++x) fetch(x, x);
        int buf = 0;
        int32_t next_share = 8;                       // tiles
        for (int32_t x = 0; x < n_stages; ++x) {
            wait_loads<(kBuffers - 2) * kLoads>();    // this wavefront's part of the stage has arrived ...
            __builtin_amdgcn_s_barrier();             // ... everyone's has, and everyone is done with the stage before
            asm volatile("" ::: "memory");
            fetch(x + kBuffers - 1, buf == 0 ? kBuffers - 1 : buf - 1);
            if (live) {
                const int32_t t0 = first_tile(x);
                if (kStage == 1) consume(buf, 0, t0, x);
                else {
                    const int m = min(kStage, n_tiles - t0);
#pragma nounroll
                    for (int i = 0; i < m; ++i) consume(buf, i, t0 + i, x * kStage + i);
                }
                if (kShares && (x + 1) * kStage >= next_share) {
                    share();
                    next_share = (x + 1) * kStage * 9 / 8 + 8;
                }
            }
            buf = buf + 1 == kBuffers ? 0 : buf + 1;
        }
        wait_loads<0>();
    }
    if (!live) return;
    if (L > 2) drain(0);

    // ---- merge the lists of a query by counting; ties to the lower part of the wavefront (the ranks are a permutation)
    int rank[L];
    float last = lk[L - 1];           // the smallest of the lists' last keys: what this query's lanes may have turned away
#pragma unroll
    for (int x = 0; x < L; ++x) rank[x] = x;
#pragma unroll
    for (int w = TILE; w < 64; w += TILE) {
        const bool before = ((lane ^ w) / TILE) < part;
        last = fminf(last, __shfl_xor(lk[L - 1], w, 64));
#pragma unroll
        for (int y = 0; y < L; ++y) {
            const float o = __shfl_xor(lk[y], w, 64);
#pragma unroll
            for (int x = 0; x < L; ++x) rank[x] += (o < lk[x] || (o == lk[x] && before)) ? 1 : 0;
        }
    }
    const int64_t p = (int64_t)q0g + qpos;
    if (L == 2) {
        // (key of rank 0 and 1 are among the lanes' entries: the second is the smallest of what is not rank 0)
#pragma unroll
        for (int x = 0; x < L; ++x) lp[x] = place_of(lp[x]);
        float best = lk[0], second = rank[0] == 0 ? lk[L - 1] : lk[0];
        int32_t bp = lp[0];
#pragma unroll
        for (int w = TILE; w < 64; w <<= 1) {
            const float ob = __shfl_xor(best, w, 64);
            const int32_t op = __shfl_xor(bp, w, 64);
            if (ob < best || (ob == best && ((lane ^ w) / TILE) < part)) { best = ob; bp = op; }
            second = fminf(second, __shfl_xor(second, w, 64));
        }
        const double eps = knn_filter_eps(P.d, fmax((double)__uint_as_float(P.Q.max_bits[grp]), (double)__uint_as_float(P.C.max_bits[grp])),
                                          kChunk * 512 / TILE);
        const bool counted = P.open_count && open_is_counted(blockIdx.x, (uint32_t)wave);
        if (kAlone || counted) {   // from the query's norm
            const float least = least_part(), longest = longest_candidate();
            const float length = ldexpf(sqrtf(P.q_norm[max(qpt, 0)]), knn_scale_exponent(P.Q.max_bits[grp])), lo = fmaf(length, 0x1p-11f, least);
            slack = 1.01f * (lo * (1.001f * longest + least) + (1.001f * length + least) * (0x1p-11f * longest + least));
        }
        const double numbers = kNumbered ? 0x1p-19 * (fabs((double)best) + fmin(fabs((double)second), 3e38)) : 0.0;   // (no second: infinity)
        const double gap = ((double)second - (double)best - numbers) * (double)key_unit, unsure = 2.0 * (double)slack * (double)key_unit;
        const bool open = qpt >= 0 && !(gap > 2.0 * eps + (kAlone ? unsure : 0.0));
        if (kNumbered && last < __builtin_inff()) last = fmaf(-0x1p-18f, fabsf(last), last);
        if (counted) {
            const unsigned long long left = __ballot(qpt >= 0 && part == 0 && !(gap > 2.0 * eps + unsure));
            if (lane == 0 && left) atomicAdd(P.open_count, (uint32_t)__popcll(left));
        }
        if (qpt >= 0 && !open && part == 0) assign.out[qpt] = knn_row(P.cmembers, c0 + (uint32_t)bp);
        const unsigned long long m = __ballot(open && part == 0);
        if (assign.open && lane == 0) assign.open[qt - P.Q.tstart[grp]] = (uint32_t)m;
        if (m == 0ull) return;
        uint32_t base = 0u;
        if (!assign.open && lane == 0) base = atomicAdd(assign.n_todo, (uint32_t)__popcll(m));
        base = __shfl(base, 0, 64);
        if (open) {
            const uint32_t slot = assign.open ? (uint32_t)p : base + (uint32_t)__popcll(m & ((1ull << (lane & (TILE - 1))) - 1ull));
            if (part == 0) { if (!assign.open) assign.todo[slot] = (int32_t)p; tau_out[slot] = (kAlone ? last - slack : last) * key_unit; }
#pragma unroll
            for (int x = 0; x < L; ++x) cand[(size_t)slot * (2 * kShare) + rank[x]] = lp[x] < 0 ? -1 : knn_row(P.cmembers, c0 + (uint32_t)lp[x]);
        }
        return;
    }
    if (qpt < 0) return;
#pragma unroll
    for (int x = 0; x < L; ++x) {
        if (rank[x] < list_len) {
            cand[p * list_len + rank[x]] = lp[x] < 0 ? -1 : knn_row(P.cmembers, c0 + (uint32_t)lp[x]);
            key_out[p * list_len + rank[x]] = lk[x] * key_unit;
        }
        if (rank[x] == list_len - 1) tau_out[p] = fminf(lk[x], last) * key_unit;
    }
}

// Wavefronts per workgroup of the filter: eight share a staged tile, unless that leaves compute units without work.  Inside clusters also as
// many as the registers allow (filter_waves): 600,000 x 64 in clusters of 4,000, k = 10, unordered, 2.82 -> 2.40 ms.  Over slices of
// the whole set eight: twelve leave fewer workgroups, and fewer of them stage the tiles, which comes out the same (7.7 ms a call).
__host__ __device__ constexpr int knn_most_waves(int tile, int steps, int L) {
    return tile == 32 ? (L == 16 ? (steps <= 2 ? 16 : steps <= 8 ? 12 : 8) : L > 16 && steps <= 2 ? 12 : 8) : L > 2 && steps <= (L == 12 ? 12 : 8) ? 12 : 8;
}
__host__ inline int knn_filter_waves(int tile, int64_t query_tiles) { return query_tiles >= 1024 ? 8 : tile == 32 ? 2 : 4; }

// list length per lane for K' = list_len candidates per query: every list longer than k (32-row tiles, two lists per query;
// a query whose k nearest all fall to one lane must still be certified), or half of K' (16-row tiles, four lists)
__host__ inline int knn_list_class(int tile, int list_len) { return tile == 32 ? (list_len <= kShortList ? 16 : 34) : list_len <= kShortList ? 12 : 20; }

// columns that the filter sums at a time for K' = list_len (1: one neighbour wanted); 0: all of them
__host__ inline int32_t knn_chunk_columns(int d, int list_len) {
    const int tile = knn_tile(d, list_len);
    return knn_chunk_steps(tile, knn_steps(d, tile), list_len == 1 ? 2 : knn_list_class(tile, list_len)) * 512 / tile;
}

}  // namespace nomad_knn
