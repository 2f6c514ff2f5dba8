// Grouped dense-layer kernels for gfx950 (MI355X): one launch runs one layer of
// every job scheduled in the round.  This is how "parallelism across lanes"
// (Salus paper, Section 3.3) is executed here: instead of one GPU stream per
// lane, the tiles of all lanes' jobs share one grid, and each workgroup finds
// its job with a ballot over the jobs' first tiles.
//
// Shape of the work: per job Y[M x N] = act(X[M x K] . W[K x N]) with M small
// (1..32 rows, more where the round is small, 64 for deep layers; the others go to kernels_gemm_tiled.hip) and
// W read straight out of the job's persistent block.  Every weight is used once per launch, so these are weight-streaming kernels.
// The four wavefronts of a workgroup split K and combine their partial tiles through LDS.  In launches that fill the chip
// W goes HBM -> registers with 16-byte loads, each wavefront keeps two k-steps of loads in flight, and the 8x8 bf16
// sub-blocks are transposed in registers into MFMA operand order.  Where a launch holds few tiles, or would load the compute units unevenly, the tiles
// are narrower and their operands go straight into an LDS ring per wavefront, for bytes in flight and not for reuse, and are transposed on
// the way out (narrow_tile.hpp).
#include <algorithm>
#include <type_traits>
#include <vector>

#include "narrow_tile.hpp"

namespace salus {

template <int MT, bool TW, bool NT>
__global__ __launch_bounds__(kGemmThreads) void grouped_dense_bf16(GroupArgs a)
{
    __shared__ float lds[reduce_lds_floats<MT * 8>()];
    Problem p;
    const Tile tile = find_tile<16 * MT, 128>(a, p);
    // A job of at most 16 rows takes the one-row-tile path even when the launch holds
    // larger jobs: its second row tile would only load clamped copies of its last row,
    // and activation loads count against the compute unit's memory path like weights do.
    if (MT == 2 && NT && p.M <= 16) dense_bf16_tile<1, TW, NT>(p, tile, lds);
    else dense_bf16_tile<MT, TW, NT>(p, tile, lds);
}

// 16 * CPL columns per workgroup, for launches with few jobs: what a launch lasts is then how long one
// compute unit streams one tile, so the tile is narrow and there are more of them.  Where every weight is read by one row
// tile (NT) its operands go straight into LDS (narrow_tile.hpp).  Transposed weights, whose lanes load 16 bytes as it
// is, and several row tiles above one another (4 jobs x 64 rows, 2048 -> 512: 7.6 us, through LDS 7.9; 16 jobs x 33 rows,
// 128 -> 512 4.0 / 4.4) keep registers.  A wavefront's k-step is only CPL / 8 of 8 KB there: deep layers keep DEEP of them
// in flight instead of two (DEEP is 0 where there are no such registers).
constexpr uint32_t kNarrowDeepK = 2048;
template <int MT, bool TW, int CPL, int DEEP, bool NT, typename Args>
__device__ inline void narrow_bf16(const Args &a)
{
    Problem p;
    if constexpr (TW || !NT) {
        __shared__ float lds[reduce_lds_floats<MT * CPL>()];
        const Tile tile = find_tile<16 * MT, 16 * CPL>(a, p);
        const bool one = MT == 2 && p.M <= 16;
        if (p.K > kNarrowDeepK) {
            if (one) dense_bf16_tile<1, TW, NT, CPL, DEEP>(p, tile, lds);
            else dense_bf16_tile<MT, TW, NT, CPL, DEEP>(p, tile, lds);
        } else {
            if (one) dense_bf16_tile<1, TW, NT, CPL>(p, tile, lds);
            else dense_bf16_tile<MT, TW, NT, CPL>(p, tile, lds);
        }
    } else {
        constexpr uint32_t kOne = NarrowTile<1, CPL>::kLds, kAll = NarrowTile<MT, CPL>::kLds;
        __shared__ __attribute__((aligned(1024))) unsigned char smem[kOne > kAll ? kOne : kAll];
        const Tile tile = find_tile<16 * MT, 16 * CPL>(a, p);
        if (MT == 2 && p.M <= 16) NarrowTile<1, CPL>::run(p, tile, smem);
        else NarrowTile<MT, CPL>::run(p, tile, smem);
    }
}

template <int MT, bool TW, int CPL, int DEEP, bool NT = true>
__global__ __launch_bounds__(kGemmThreads) void grouped_dense_bf16_narrow(GroupArgs a) { narrow_bf16<MT, TW, CPL, DEEP, NT>(a); }
template <int MT, bool TW, int CPL, int DEEP, bool NT = true>
__global__ __launch_bounds__(kGemmThreads) void grouped_dense_bf16_narrow(FewArgs a) { narrow_bf16<MT, TW, CPL, DEEP, NT>(a); }

// Tiles of 64, 80, 96 or 128 columns, operands through LDS, two workgroups per compute unit: for launches of too many jobs for narrow
// tiles whose 128-column tiles would leave compute units unevenly loaded (even_columns).  48 jobs x 1 - 32 rows,
// 3080 -> 776, weights from HBM: 48.9 us with 80 columns (480 tiles), 58.6 with 128 through registers (336).
template <int MT, int NB>
__global__ __launch_bounds__(kGemmThreads, 2) void grouped_dense_bf16_even(GroupArgs a)
{
    using One = NarrowTile<1, NB, 1, 80 * 1024>;
    using All = NarrowTile<MT, NB, 1, 80 * 1024>;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[One::kLds > All::kLds ? One::kLds : All::kLds];
    Problem p;
    const Tile tile = find_tile<16 * MT, 16 * NB>(a, p);
    if (MT == 2 && p.M <= 16) One::run(p, tile, smem);
    else All::run(p, tile, smem);
}

// 64-row tiles of 128 columns for deep layers of jobs with 33 .. 64 rows: every weight passes through a
// compute unit once.  Two workgroups per compute unit (registers capped accordingly), so that one
// workgroup's reduction and epilogue overlap the other's stream.
__global__ __launch_bounds__(kGemmThreads, 2) void grouped_dense_bf16_rows64(GroupArgs a)
{
    __shared__ float lds[reduce_lds_floats<32>()];
    Problem p;
    const Tile tile = find_tile<64, 128>(a, p);
    dense_bf16_tile<4, false, true>(p, tile, lds);
}

// Row tiles of 16 * MT rows; the last one of a job computes only as many 16-row blocks as it needs (the sums of a row do not
// depend on how many there are).  A single block has little to multiply between its loads: three k-steps in flight instead of
// two (12 jobs x 16 rows, 516 -> 1204, two / three / four / six: 8.6 / 6.0 / 6.3 / 6.6 us; 5 jobs x 16 rows, 900 -> 1500, three 7.7, four 8.1).
template <int MT, typename Args>
__device__ inline void rows_f32(const Args &a)
{
    __shared__ float lds[reduce_lds_floats<MT * 4>()];
    Problem p;
    const Tile tile = find_tile<16 * MT, 64>(a, p);
    const uint32_t rows = p.M - tile.m0;
    if (MT == 1 || rows <= 16) dense_f32_tile<1, 3>(p, tile, lds);
    else if (MT > 2 && rows <= 32) dense_f32_tile<2>(p, tile, lds);
    else dense_f32_tile<MT>(p, tile, lds);
}

template <int MT>
__global__ __launch_bounds__(kGemmThreads) void grouped_dense_f32(GroupArgs a) { rows_f32<MT>(a); }
template <int MT>
__global__ __launch_bounds__(kGemmThreads) void grouped_dense_f32(FewArgs a) { rows_f32<MT>(a); }

// The same for 16-row tiles, four k-steps in flight: for wavefronts of five or eight steps, or twelve more, which end with a batch of two where three are in flight, and, if weights come
// from HBM, of four.  Four / three, from the cache and from HBM: 82 jobs x 2 rows, 276 -> 944, 19.8 / 24.5 and 20.3 / 25.6 us, 30 jobs x 16 rows, 320 -> 1024, 9.1 / 11.6 and 9.6 / 11.9.  Over
// seven sets of jobs, by steps: 5 0.99 and 0.95 of the time, 8 0.99 and 0.96, 17 1.00 and 0.985, 20 1.00 and 0.98, 4 1.02 and 0.97; 2, 3, 6, 7, 10, 11, 15, 18, 19 1.02 - 1.07 and
// 1.02 - 1.07, the others 1.00 - 1.02 and 0.99 - 1.01.
template <typename Args>
struct FourInFlight : Args {};      // names this variant of the kernel
template <int MT, typename Args>
__device__ inline void four_in_flight_f32(const Args &a)
{
    static_assert(MT == 1, "16-row tiles");
    __shared__ float lds[reduce_lds_floats<4>()];
    Problem p;
    const Tile tile = find_tile<16, 64>(a, p);
    dense_f32_tile<1, 4>(p, tile, lds);
}

template <int MT>
__global__ __launch_bounds__(kGemmThreads) void grouped_dense_f32(FourInFlight<GroupArgs> a) { four_in_flight_f32<MT>(a); }
template <int MT>
__global__ __launch_bounds__(kGemmThreads) void grouped_dense_f32(FourInFlight<FewArgs> a) { four_in_flight_f32<MT>(a); }

// 16 columns and 16 rows per workgroup, for launches of few tiles: a launch lasts as long as one wavefront's chain of
// multiplies and loads over its quarter of K, and this tile has a quarter of the multiplies.  16 columns / 64, 4 jobs x 16 rows, 1536 ->
// 1000: 6.7 / 10.7 us, 1024 -> 1000 5.5 / 8.0, 384 -> 1000 4.1 / 5.2 on the device, 2 jobs x 8 rows, 256 -> 256 3.4 / 4.4.
template <typename Args>
__device__ inline void narrow_f32(const Args &a)
{
    __shared__ float lds[reduce_lds_floats<1>()];
    Problem p;
    const Tile tile = find_tile<16, 16>(a, p);
    dense_f32_tile<1, 4, 1>(p, tile, lds);
}

__global__ __launch_bounds__(kGemmThreads) void grouped_dense_f32_narrow(GroupArgs a) { narrow_f32(a); }
__global__ __launch_bounds__(kGemmThreads) void grouped_dense_f32_narrow(FewArgs a) { narrow_f32(a); }

// ---------------------------------------------------------------------------
// force_mt != 0: row tiles of 16 * force_mt rows whatever the jobs' sizes.  Launch: called with FewArgs where it takes them and they suffice.
template <typename Launch>
static hipError_t launch_groups(const Problem *p, uint32_t n, uint32_t tn, uint32_t m_small,
                                uint32_t m_mid, Launch launch, uint64_t *launches, int force_mt = 0)
{
    for (uint32_t at = 0; at < n; at += kMaxProblems) {
        const uint32_t count = std::min(kMaxProblems, n - at);
        uint32_t max_m = 0;
        for (uint32_t i = 0; i < count; ++i) max_m = std::max(max_m, p[at + i].M);
        const int mt = force_mt ? force_mt : max_m <= m_small ? 1 : max_m <= m_mid ? 2 : 4;
        const uint32_t tm = 16u * mt;
        auto go = [&](auto &&a) {
            const uint64_t tiles = fill_group(a, p + at, count, [&](const Problem &q) { return (uint64_t)((q.M + tm - 1) / tm) * ((q.N + tn - 1) / tn); });
            if (tiles == 0) return hipSuccess;
            if (tiles > 0x7fffffffull) return hipErrorInvalidValue;
            launch(mt, a, (uint32_t)tiles);
            if (launches) *launches += 1;
            return hipGetLastError();
        };
        hipError_t e;
        if constexpr (std::is_invocable_v<Launch, int, const FewArgs &, uint32_t>) e = count <= kFewProblems ? go(FewArgs{}) : go(GroupArgs{});
        else e = go(GroupArgs{});
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Rows per job from which the LDS-tiled kernel is used: always from 128 rows; from
// 65 rows if the jobs routed there make up at least one workgroup per CU (256).
constexpr uint32_t kTiledAlways = 128, kTiledMaybe = 65;
constexpr uint64_t kTiledMinGrid = 256;
constexpr uint64_t kMixedMinGrid = 96;   // 128 x 256 tiles
constexpr uint64_t kFullGrid = 256;      // one workgroup per compute unit
constexpr uint32_t kDeepK = 1024;

// Tile width (in 16 columns) with which the busiest compute unit streams least, its weights and the activations beside them; 0: 128
// columns through registers.  What the change is worth depends on the rows of the weights and on where they come from.
// Whole lines: 80 columns cost a fifth more and 96 a third (8 jobs, 3072 -> 2688, 96 columns 1.3 of 128), so those never pay.  From the
// cache (256 MB) where the load falls by a tenth, but with one tile of 128 per compute unit not in shallow layers (40 jobs, 768
// wide, three layers 30 / 32 us); 128 columns through LDS there only for jobs of 17 rows and more, in layers deeper than 2048 with at most three
// tiles for four compute units and in those deeper than 3072 (registers / LDS, up to 16 rows: 47 jobs, 1152 -> 512 9.9 / 10.9, 24 jobs, 1152 -> 1152
// 0.90, 9 jobs, 1536 -> 2688 0.94; 26 jobs, 2496 -> 832 (182 tiles) 1.12, 21 jobs, 2176 -> 960 (168) 1.08, 50 jobs, 2176 -> 640 (250) 0.96, 27 jobs, 2688 -> 1024
// (216) 0.96; 42 jobs, 3136 -> 576 (210) 1.09, 23 jobs, 3328 -> 1024 1.07; 32 rows: 20 jobs, 1664 -> 1408 0.99, 23 jobs, 2944 -> 1024 1.14).  From HBM only where 64 columns nearly halve
// the load (45 jobs, 2560 -> 320: 18.2 / 14.9; at 0.8 of the load 12 jobs, 1792 -> 1536 0.92; 20 jobs x 1 - 32 rows, 2048 -> 2048 -> 2048 -> 2048, strips: 102 / 111).
// Rows that begin inside a line, which cost registers extra: from the cache always (17 jobs, 472 -> 1712, the same load either way 6.4 / 5.1, 64
// jobs x 32 rows, 680 -> 1760, 1.16, 33 jobs, 2832 -> 928 45 / 28), in layers below 320 where the load falls by a fifth (28 jobs, 136 -> 928, 64 jobs,
// 256 -> 424, the same load 0.90 and 0.92, 184 -> 1560, 0.83 of it 0.91, 30 jobs, 224 -> 1464, 0.78 of it 1.26).  From HBM where it falls by a tenth (40
// jobs, 776 wide, nine layers 156 / 140 us, 16 jobs, 3080 -> 1496 -> 3080 -> 1496 101 / 88; without: 24 jobs, 1160 wide, 107 / 122), in layers below 512
// by three tenths (21 jobs, 424 -> 3752, 0.89 of the load 15.0 / 16.3, 59 jobs, 296 -> 1096, 0.79 of it 13.3 / 14.8, 10 jobs, 384 -> 3304, 0.67 of it 1.08).
static uint32_t even_columns(const Problem *p, uint32_t n, bool cached)
{
    uint64_t two = 0, wide_tiles = 0;
    uint32_t min_k = ~0u, max_k = 0;
    bool lines = true;
    for (uint32_t i = 0; i < n; ++i) {
        const Problem &q = p[i];
        two += q.M > 16;
        min_k = std::min(min_k, q.K);
        max_k = std::max(max_k, q.K);
        lines = lines && ((q.flags & kStripW) || q.N % 64 == 0);
        wide_tiles += (q.N + 127) / 128;
    }
    const bool one_each = wide_tiles <= kFullGrid;
    if (lines && cached && min_k <= kDeepK && one_each) return 0;
    const uint64_t x = two * 2 > n ? 20 : two ? 15 : 10;      // tenths of what 16 columns of weights are
    auto cost = [&](uint64_t tiles, uint32_t nb) { return (tiles + kFullGrid - 1) / kFullGrid * (10 * nb + x) * (lines && nb == 5 ? 12 : 10); };
    // in tenths of what registers take
    const uint32_t at_most = lines ? (!cached ? 6 : one_each ? 10 : 9) : cached ? (max_k < 320 ? 8 : 100) : max_k < 512 ? 7 : 9;
    const uint32_t lds_from = wide_tiles * 4 <= kFullGrid * 3 ? 2 * kDeepK : 3 * kDeepK;
    uint64_t least = cost(wide_tiles, 8) * at_most / 10;
    uint32_t best = 0;
    for (const uint32_t nb : {8u, 4u, 5u, 6u}) {
        if (lines && (nb == 6 || (nb == 8 && min_k <= lds_from && !two))) continue;
        uint64_t tiles = 0;
        for (uint32_t i = 0; i < n; ++i) tiles += (p[i].N + 16 * nb - 1) / (16 * nb);
        const uint64_t c = cost(tiles, nb);
        if (c > least || (c == least && best)) continue;
        least = c;
        best = nb;
    }
    return best;
}

static uint64_t count_tiles(const Problem *p, uint32_t n, uint32_t tm, uint32_t tn)
{
    uint64_t tiles = 0;
    for (uint32_t i = 0; i < n; ++i) tiles += (uint64_t)((p[i].M + tm - 1) / tm) * ((p[i].N + tn - 1) / tn);
    return tiles;
}

// Columns of 32-row register tiles, several above one another, of which there is at most one per compute unit: 32, 64 or 0.
static uint32_t narrow_columns(const Problem *p, uint32_t n)
{
    return count_tiles(p, n, 32, 64) > kFullGrid ? 0 : count_tiles(p, n, 32, 32) <= kFullGrid ? 32 : 64;
}

static hipError_t launch_narrow_rows(const Problem *p, uint32_t n, bool trans_w, uint32_t columns, hipStream_t stream, uint64_t *launches)
{
    auto launch = [&](int, const auto &a, uint32_t tiles) {
        const dim3 grid(tiles), block(kGemmThreads);
        if (trans_w) hipLaunchKernelGGL((grouped_dense_bf16_narrow<2, true, 2, 8, false>), grid, block, 0, stream, a);
        else if (columns == 32) hipLaunchKernelGGL((grouped_dense_bf16_narrow<2, false, 2, 8, false>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((grouped_dense_bf16_narrow<2, false, 4, 4, false>), grid, block, 0, stream, a);
    };
    return launch_groups(p, n, columns, 0, 0, launch, launches, 2);
}

// Jobs of 128 rows and more whose large tiles would leave most compute units idle, in layers deeper than five slabs: the smallest tile of which
// there is at most one per compute unit, 32 x 32 and 32 x 64 through registers, 64 x 64 and 64 x 128 through the ring; and 64 x 128, two
// per compute unit, where 128 x 128 tiles would be between one and two.  Before (128 x 128 or larger) / now: 1 job x 260 rows, 3200 -> 448, 28.3 / 10.1 us,
// 1 job x 463 rows, 1024 -> 920, 12.4 / 6.8, 4 jobs x 129 rows, 1536 -> 1024, 16.8 / 9.6, 4 jobs x 429 rows, 1792 -> 1056, 19.8 /
// 14.3, 6 jobs x 168 rows, 3392 -> 2944, 41.0 / 35.5.  Over 95 such launches with weights from the cache 0.57 of the time before on
// average and 0.93 at most, within 3 % of the quickest of seven kinds of tiles in all but two; over 40 drawn ones 0.58, and 0.63 (0.95 at most) with
// weights from HBM.  Tiles beyond one per compute unit: 4 jobs x 619 rows, 320 -> 576, 32 x 64 8.8 us, 64 x 64 6.1.
// Two limits do not lie where the times cross.  Layers of 320 and rounds that hold jobs of 128 rows among larger ones (a launch of large tiles for each height) keep
// what they had and would gain too, large / these tiles: 1 job x 256 rows, 320 -> 4096, 8.1 / 5.4 us, 5 jobs x 268, 320 -> 2392, 11.2 / 9.2; one job x 128 rows and one
// x 256, 1024 -> 1024, 25.2 / 6.9, 128, 333 and 600 rows, 512 -> 320, 17.5 / 5.0.
static bool few_tiles(const Problem *p, uint32_t n)
{
    uint32_t of_128 = 0;
    for (uint32_t i = 0; i < n; ++i) {
        if (p[i].M < kTiledAlways || p[i].K < 384) return false;
        of_128 += p[i].M == kTiledAlways;
    }
    if (of_128 != 0 && of_128 != n) return false;
    const uint64_t tiles = count_tiles(p, n, 64, 128);
    return tiles <= kFullGrid || (tiles <= 2 * kFullGrid && count_tiles(p, n, 128, 128) > kFullGrid);
}

hipError_t launch_grouped_bf16(const Problem *p, uint32_t n, bool trans_w, bool cached, hipStream_t stream,
                               uint64_t *launches)
{
    // Jobs with many rows reuse every weight often enough to pay for LDS staging:
    // they go to the tiled kernel, the rest of the round to the streaming kernel.
    // (A round of small jobs takes less time on the device than on the host: no lists are built that it does not need.)
    uint32_t max_m = 0;
    for (uint32_t i = 0; i < n; ++i) max_m = std::max(max_m, p[i].M);
    if (!trans_w && max_m > 32) {
        uint64_t grid = 0;
        for (uint32_t i = 0; i < n; ++i)
            if (p[i].M >= kTiledMaybe && tiled_shape_ok(p[i])) grid += tiled_tiles(p[i]);
        const uint32_t min_m = grid >= kTiledMinGrid ? kTiledMaybe : kTiledAlways;
        // Deep layers of a round that mixes jobs of 33 .. 64 and of 65 .. 128 rows: all in one launch of the tiled kernel from
        // 96 tiles of 128 x 256 (the 128 x 128 ones it may take instead then hold most compute units), below that through
        // the ring.  Tiled / ring, 30 jobs x 33 - 87 rows, 3584 -> 1536 (180 tiles): 77 / 92 us, 1584 -> 776 (120): 28 / 36,
        // 1536 -> 768 (90): 27 / 25; 20 jobs x 33 - 128 rows, 4096 -> 1024 (80): 55 / 47.  Two launches, one for each range
        // of rows, never: 116, 52 and 47 us for the first three.  (64 models x 33 - 128 rows, 4096 -> 1024 / 1024 -> 4096 / 1024 -> 1024: 112 / 134 / 39 us against
        // 149 / 149 / 45 us with 64-row tiles, whose second row tile reads the weights again).
        uint64_t mid_grid = 0;
        bool above_64 = false;
        auto deep_mid = [](const Problem &q) { return q.M > 32 && q.M <= 128 && q.K >= kDeepK && tiled_shape_fits(q); };
        for (uint32_t i = 0; i < n; ++i)
            if (deep_mid(p[i])) {
                mid_grid += tiled_tiles(p[i]);
                above_64 = above_64 || p[i].M > 64;
            }
        const bool take_mid = above_64 && mid_grid >= kMixedMinGrid;
        // Jobs whose K is no multiple of a slab or at most 256: all of them in the tiled kernel if they hold more than two
        // 32-row register tiles per compute unit (deeper than 2048: 1.25), else none: register tiles split K over wavefronts
        // where a compute unit would walk a large tile alone.  Register / tiled, 1 job x 256 rows, 3080 -> 776 (56 register
        // tiles): 17.6 / 27.9 us, 1032 -> 72 8.0 / 12.4; 8 jobs x 129 rows, 776 -> 1016 (320) 10.9 / 11.6, 16 jobs (640) 17.4 / 13.0; 4 jobs x
        // 600 rows, 3080 -> 776 (532) 46.6 / 31.1; depths of 64 - 256, up to 512 tiles 0.36 - 1.00 of tiled, from 640 1.2 - 3.
        // The rows do not matter beside that, and one rule for all of them keeps a round in one launch: 8 jobs x 100 - 400 rows,
        // 1000 -> 3080 -> 776, 81 us against 111 us when those from 192 rows went to the tiled kernel and the others did not.
        // Beside jobs that take the tiled kernel anyway they join those, again for one launch; so do shallow ones with rows on
        // either side of 192, which have a launch for each tile height.
        bool shallow_low = false, shallow_high = false;
        for (uint32_t i = 0; i < n; ++i)
            if (p[i].M >= min_m && tiled_shape_ok(p[i]) && tiled_shape_shallow(p[i]))
                (p[i].M >= kTiled256MinM ? shallow_high : shallow_low) = true;
        const bool both = shallow_low && shallow_high;
        auto always = [&](const Problem &q) { return q.M >= min_m && tiled_shape_ok(q) && (both || !tiled_shape_shallow(q)); };
        auto if_many = [&](const Problem &q) {
            return tiled_shape_ragged(q) || (!both && q.M >= min_m && tiled_shape_ok(q) && tiled_shape_shallow(q));
        };
        uint64_t many_tiles = 0;
        bool many_deep = true, tiled_anyway = false;
        for (uint32_t i = 0; i < n; ++i)
            if (always(p[i])) tiled_anyway = true;
            else if (if_many(p[i])) {
                many_tiles += (uint64_t)((p[i].M + 31) / 32) * ((p[i].N + 127) / 128);
                many_deep = many_deep && p[i].K > kNarrowDeepK;
            }
        const bool many = tiled_anyway || many_tiles > (many_deep ? kFullGrid * 5 / 4 : kFullGrid * 2);
        auto takes_tiled = [&](const Problem &q) { return always(q) || (take_mid && deep_mid(q)) || (many && if_many(q)); };
        if (std::any_of(p, p + n, takes_tiled)) {
            std::vector<Problem> tiled, streamed;
            for (uint32_t i = 0; i < n; ++i) (takes_tiled(p[i]) ? tiled : streamed).push_back(p[i]);
            const uint32_t count = (uint32_t)tiled.size();
            const bool few = few_tiles(tiled.data(), count);
            const uint32_t columns = few ? narrow_columns(tiled.data(), count) : 0;
            hipError_t e = columns ? launch_narrow_rows(tiled.data(), count, false, columns, stream, launches)
                           : few   ? launch_grouped_bf16_stream(tiled.data(), count, false, true, stream, launches)
                                   : launch_grouped_bf16_tiled(tiled.data(), count, cached, stream, launches);
            if (e != hipSuccess || streamed.empty()) return e;
            return launch_grouped_bf16(streamed.data(), (uint32_t)streamed.size(), false, cached, stream, launches);
        }
    }
    // Up to 32 rows: one row tile of 16 or 32 rows per job, 128 columns, every weight read once (non-temporal).
    // 33 .. 128 rows (those the tiled kernel did not take): 64-row tiles fed through an LDS ring
    // (launch_grouped_bf16_stream), except that deep layers of at least 1024 of jobs of up to 64 rows, with enough jobs
    // to fill the chip, keep one 64-row tile of 128 columns straight from memory (64 models at 64 rows, 4096 -> 1024 /
    // 1024 -> 4096 / 1024 -> 1024: 115 / 125 / 33 us against 117 / 130 / 34 us through the ring); registers are capped
    // for two workgroups per compute unit there, without which it was slower.  Above 128 rows transposed weights take
    // the ring as well (input gradients of 4 jobs x 500 rows, 2048 -> 2048: 40 us against 77 us with 32-row tiles; the
    // 128 x 128 tiles of the compute-bound kernel are within 2 % at 500 and 1024 rows and slower below); forward layers come
    // here only if they are too few or too shallow for the tiled kernel, and get 32-row tiles.
    std::vector<Problem> small, mid, large;
    (max_m <= 32 ? small : mid).reserve(n);
    for (uint32_t i = 0; i < n; ++i) {
        const bool ring = tiled_shape_fits(p[i]);
        (p[i].M <= 32 ? small : ring && (p[i].M <= 128 || trans_w) ? mid : large).push_back(p[i]);
    }
    uint64_t small_tiles = 0;
    for (const Problem &q : small) small_tiles += (q.N + 127) / 128;
    if (trans_w && small_tiles * 4 > kFullGrid) {
        // Input gradients of 17 .. 32 rows take the ring too, unless 32-column tiles do (below).  Training step, 8 jobs x 32
        // rows, 2048-wide layers: 360 us against 375; 2 jobs x 24 rows: 146 against 140, so not there.
        std::vector<Problem> rest;
        for (const Problem &q : small) (q.M > 16 && tiled_shape_fits(q) ? mid : rest).push_back(q);
        small.swap(rest);
    }
    auto launch_wide = [&](int mt, const GroupArgs &a, uint32_t tiles) {
        const dim3 grid(tiles), block(kGemmThreads);
        bool one_row_tile = true;      // else several row tiles read the same weights: plain loads, L2 serves the others
        for (uint32_t i = 0; i < a.n; ++i) one_row_tile = one_row_tile && a.p[i].M <= 16u * mt;
        if (mt == 4) hipLaunchKernelGGL(grouped_dense_bf16_rows64, grid, block, 0, stream, a);
        // (transposed weights with several row tiles: only widths from 2^22, which the ring cannot address)
        else if (!one_row_tile && trans_w) hipLaunchKernelGGL((grouped_dense_bf16<2, true, false>), grid, block, 0, stream, a);
        else if (!one_row_tile) hipLaunchKernelGGL((grouped_dense_bf16<2, false, false>), grid, block, 0, stream, a);
        else if (mt == 2 && trans_w) hipLaunchKernelGGL((grouped_dense_bf16<2, true, true>), grid, block, 0, stream, a);
        else if (mt == 2) hipLaunchKernelGGL((grouped_dense_bf16<2, false, true>), grid, block, 0, stream, a);
        else if (trans_w) hipLaunchKernelGGL((grouped_dense_bf16<1, true, true>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((grouped_dense_bf16<1, false, true>), grid, block, 0, stream, a);
    };
    // Every launch of up to kMaxProblems jobs for itself: what counts is how its own tiles spread over the compute units (100 jobs,
    // 1024 -> 200, are launches of 128 and 72 tiles, not one of 200).
    for (uint32_t at = 0; at < small.size(); at += kMaxProblems) {
        const Problem *q = small.data() + at;
        const uint32_t count = std::min(kMaxProblems, (uint32_t)small.size() - at);
        uint64_t tiles_128 = 0;
        for (uint32_t i = 0; i < count; ++i) tiles_128 += (q[i].N + 127) / 128;
        const bool fits = std::all_of(q, q + count, tiled_shape_fits), narrow = tiles_128 * 2 <= kFullGrid && (trans_w || fits);
        const uint32_t nb = trans_w || narrow || !fits ? 0 : even_columns(q, count, cached);
        auto launch_even = [&](int mt, const GroupArgs &a, uint32_t tiles) {
            auto go = [&](auto one, auto two) { hipLaunchKernelGGL(mt == 2 ? two : one, dim3(tiles), dim3(kGemmThreads), 0, stream, a); };
            if (nb == 4) go(grouped_dense_bf16_even<1, 4>, grouped_dense_bf16_even<2, 4>);
            else if (nb == 5) go(grouped_dense_bf16_even<1, 5>, grouped_dense_bf16_even<2, 5>);
            else if (nb == 6) go(grouped_dense_bf16_even<1, 6>, grouped_dense_bf16_even<2, 6>);
            else go(grouped_dense_bf16_even<1, 8>, grouped_dense_bf16_even<2, 8>);
        };
        // As many workgroups as compute units, not more: a narrower tile streams less efficiently.  32 / 16 columns, one job x
        // 1 row: 2048 -> 1024 4.9 / 4.0 us (32 / 64 workgroups; 32 columns through registers 9.2), 1024 -> 1024 3.6 / 3.2, x 32 rows
        // 5.1 / 4.8, 4 jobs x 32 rows 5.3 / 5.0.  Transposed weights, 128 / 64 / 32 columns: 2048 -> 2048 of 4 jobs 20.3 /
        // 16.2 / 14.5, of 8 jobs 18.3 / 15.5 / 20.9, of 16 jobs 25.6 / 28.8 / 43.6.  (Widths from 2^22, which the direct-to-LDS
        // loads cannot address, keep 128.)
        auto launch_16 = [&](int mt, const auto &a, uint32_t tiles) {
            const dim3 grid(tiles), block(kGemmThreads);
            if (mt == 2) hipLaunchKernelGGL((grouped_dense_bf16_narrow<2, false, 1, 0>), grid, block, 0, stream, a);
            else hipLaunchKernelGGL((grouped_dense_bf16_narrow<1, false, 1, 0>), grid, block, 0, stream, a);
        };
        auto launch_64 = [&](int mt, const auto &a, uint32_t tiles) {
            const dim3 grid(tiles), block(kGemmThreads);
            if (mt == 2 && trans_w) hipLaunchKernelGGL((grouped_dense_bf16_narrow<2, true, 4, 4>), grid, block, 0, stream, a);
            else if (mt == 2) hipLaunchKernelGGL((grouped_dense_bf16_narrow<2, false, 4, 0>), grid, block, 0, stream, a);
            else if (trans_w) hipLaunchKernelGGL((grouped_dense_bf16_narrow<1, true, 4, 4>), grid, block, 0, stream, a);
            else hipLaunchKernelGGL((grouped_dense_bf16_narrow<1, false, 4, 0>), grid, block, 0, stream, a);
        };
        auto launch_32 = [&](int mt, const auto &a, uint32_t tiles) {
            const dim3 grid(tiles), block(kGemmThreads);
            if (mt == 2 && trans_w) hipLaunchKernelGGL((grouped_dense_bf16_narrow<2, true, 2, 8>), grid, block, 0, stream, a);
            else if (mt == 2) hipLaunchKernelGGL((grouped_dense_bf16_narrow<2, false, 2, 0>), grid, block, 0, stream, a);
            else if (trans_w) hipLaunchKernelGGL((grouped_dense_bf16_narrow<1, true, 2, 8>), grid, block, 0, stream, a);
            else hipLaunchKernelGGL((grouped_dense_bf16_narrow<1, false, 2, 0>), grid, block, 0, stream, a);
        };
        const hipError_t e = nb                                         ? launch_groups(q, count, 16 * nb, 16, 32, launch_even, launches)
                             : !narrow                                  ? launch_groups(q, count, 128, 16, 32, launch_wide, launches)
                             : !trans_w && tiles_128 * 8 <= kFullGrid   ? launch_groups(q, count, 16, 16, 32, launch_16, launches)
                             : tiles_128 * 4 <= kFullGrid               ? launch_groups(q, count, 32, 16, 32, launch_32, launches)
                                                                        : launch_groups(q, count, 64, 16, 32, launch_64, launches);
        if (e != hipSuccess) return e;
    }
    if (!mid.empty()) {
        // Too few for the ring, whose workgroup walks all of K in a row of slabs: narrow 32-row tiles as above, K split over
        // the wavefronts, as many workgroups as compute units.  Ring / narrow, one job x 33 rows, 1024 -> 64: 8.5 / 5.2 us
        // (the 64 x 64 register tile that the ring replaced: 7.1), 4096 -> 1024 20.4 / 11.9 (16.5); 16 jobs x 33 rows,
        // 128 -> 512, 64 columns: 6.1 / 4.5 (5.7); 10 jobs x 33 rows, 1024 -> 512 9.0 / 7.3 (7.8); beyond one per compute unit,
        // 24 jobs x 65 rows, 1024 -> 512: 11.0 / 14.1.
        // Input gradients take those of 32 columns only: steps of 2 jobs x 43 rows of 544 - 632 - 856 - 1704 - 240 58.5 us with them and 63.4 through the
        // ring, 1 job x 147 rows of 1616 - 856 - 536 - 1192 - 128 69.6 / 73.9; with 64 columns too 1 job x 344 rows of 672 - 1384 - 856 - 832 - 896 77.2 / 75.0.
        const uint32_t columns = narrow_columns(mid.data(), (uint32_t)mid.size());
        if (columns == 32 || (columns && !trans_w)) {
            if (hipError_t e = launch_narrow_rows(mid.data(), (uint32_t)mid.size(), trans_w, columns, stream, launches)) return e;
            mid.clear();
        }
    }
    if (!mid.empty()) {
        uint64_t wide_tiles = 0;
        bool mixed = false;      // one launch for jobs below and above 64 rows
        for (const Problem &q : mid) {
            wide_tiles += (uint64_t)((q.M + 63) / 64) * ((q.N + 127) / 128);
            mixed = mixed || q.M > 64;
        }
        const bool full = wide_tiles >= kFullGrid && !trans_w && !mixed;
        std::vector<Problem> deep, ring;
        if (full)
            for (const Problem &q : mid) (q.K >= kDeepK ? deep : ring).push_back(q);
        else ring.swap(mid);
        if (!ring.empty())
            if (hipError_t e = launch_grouped_bf16_stream(ring.data(), (uint32_t)ring.size(), trans_w, false, stream, launches)) return e;
        if (!deep.empty())
            if (hipError_t e = launch_groups(deep.data(), (uint32_t)deep.size(), 128, 0, 0, launch_wide, launches, 4)) return e;
    }
    if (!large.empty())
        if (hipError_t e = launch_groups(large.data(), (uint32_t)large.size(), 128, 0, 0, launch_wide, launches, 2)) return e;
    return hipSuccess;
}

hipError_t launch_grouped_f32(const Problem *p, uint32_t n, bool cached, hipStream_t stream, uint64_t *launches)
{
    auto launch = [&](int mt, const auto &a, uint32_t tiles) {
        const bool four = std::all_of(a.p, a.p + a.n, [&](const Problem &q) {
            const uint32_t steps = (q.K + 63) / 64;      // of 16 k-rows, a wavefront's share of them
            return steps % 12 == 5 || steps % 12 == 8 || (steps == 4 && !cached);
        });
        if (mt == 1 && four)
            hipLaunchKernelGGL(grouped_dense_f32<1>, dim3(tiles), dim3(kGemmThreads), 0, stream, FourInFlight<std::decay_t<decltype(a)>>{a});
        else if (mt == 1)
            hipLaunchKernelGGL(grouped_dense_f32<1>, dim3(tiles), dim3(kGemmThreads), 0, stream, a);
        else if (mt == 2)
            hipLaunchKernelGGL(grouped_dense_f32<2>, dim3(tiles), dim3(kGemmThreads), 0, stream, a);
        else
            hipLaunchKernelGGL(grouped_dense_f32<4>, dim3(tiles), dim3(kGemmThreads), 0, stream, a);
    };
    // Float multiplies are what a 64-row tile takes long for (16 x 16 x 4 per instruction), so rows are spread over
    // workgroups.  16-row tiles as long as two per compute unit hold them, except that 32-row tiles take layers deeper than 256 of which there are more than one
    // 16-row tile per compute unit and no more than one of those: two 16-row tiles on a compute unit read the weights twice (12 jobs x 1 - 77 rows, 1204 ->
    // 780, 273 / 208 tiles: 17.3 / 13.8 us, with weights from HBM 24.0 / 18.1; 5 jobs x 86 rows, 1012 -> 936, 14.1 / 12.2 and 17.6 / 13.6; over 32 such
    // layers 0.94 and 0.86 of the time; 4 jobs x 52 rows, 200 -> 976 5.1 / 5.2; more than one 32-row tile per compute unit: 8 jobs x 68 rows, 988 -> 760, 13.7 / 20.2).  Else 64-row tiles while those leave compute units idle,
    // or if they fill whole rounds of the chip and every job has the rows for them (a weight is then read half as often); else
    // 32-row tiles.  16 / 32 / 64 rows per tile: the layers of 12 jobs x 1 - 128 rows, 516 -> 1204 -> 780 -> 388: 10.9 / 15.1 / 19.8,
    // 17.2 / 15.6 / 26.4 and 6.8 / 10.3 / 17.3 us; one job x 64 rows, 1024 -> 1024 8.0 / 11.9 / 20.4; 12 jobs x 32 rows, 1204 -> 780 (312 16-row tiles) 16.6 / 15.1, 40 jobs, 256 -> 256
    // (320) 5.6 / 5.6; 12 jobs x 128 rows, 1536 -> 1536 81 / 73 / 86, 4 jobs 27 / 30 / 29 (from HBM 32 / 32 / 30); 40 jobs x 33 rows, 1536 -> 1536 (960 64-row tiles, 3.75
    // rounds), 32 / 64 rows: 122 / 111; 40 jobs x 128 rows, 1024 -> 1024 (5 rounds) 92 / 93, 40 rows (2.5) 53 / 57.
    uint64_t tiles_16 = 0, tiles_32 = 0, tiles_64 = 0;
    uint32_t max_m = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const uint64_t cols = (p[i].N + 63) / 64;
        tiles_16 += (p[i].M + 15) / 16 * cols;
        tiles_32 += (p[i].M + 31) / 32 * cols;
        tiles_64 += (p[i].M + 63) / 64 * cols;
        max_m = std::max(max_m, p[i].M);
    }
    const uint64_t rounds_64 = (tiles_64 + kFullGrid - 1) / kFullGrid;
    const bool whole_64 = tiles_32 == 2 * tiles_64 && tiles_64 * 16 >= rounds_64 * kFullGrid * 15;
    const int mt = tiles_16 <= 2 * kFullGrid                       ? 1
                   : max_m > 128 || tiles_64 <= kFullGrid          ? 0
                   : max_m > 32 && whole_64                        ? 4
                   : max_m > 16                                    ? 2 : 1;
    // One 32-row tile per compute unit, and 16 columns as long as there is at most one such tile per compute unit, in every launch for itself: 90 jobs x
    // 48 rows, 900 -> 64, are launches of 192 and 78 16-row tiles, not one of 270 (15.0 us, with 32 rows 22.7); 6 jobs x 16 rows, 1024 -> 1024 (384), 16 / 64
    // columns 7.6 / 7.9 us, 12 jobs (768) 12.7 / 10.9.
    auto launch_narrow = [&](int, const auto &a, uint32_t tiles) {
        hipLaunchKernelGGL(grouped_dense_f32_narrow, dim3(tiles), dim3(kGemmThreads), 0, stream, a);
    };
    for (uint32_t at = 0; at < n; at += kMaxProblems) {
        const uint32_t count = std::min(kMaxProblems, n - at);
        const Problem *q = p + at;
        const bool deep = std::all_of(q, q + count, [](const Problem &r) { return r.K > 256; });
        const bool one_32 = deep && count_tiles(q, count, 16, 64) > kFullGrid && count_tiles(q, count, 32, 64) <= kFullGrid;
        const hipError_t e = count_tiles(q, count, 16, 16) <= kFullGrid ? launch_groups(q, count, 16, 0, 0, launch_narrow, launches, 1)
                                                                        : launch_groups(q, count, 64, 16, 32, launch, launches, one_32 ? 2 : mt);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace salus
