// Grouped dense layer for jobs that bring many rows: the compute-bound counterpart of the weight-streaming
// kernels.  Same contract (one launch runs one layer of every scheduled job, Salus paper, Section 3.3), but
// here a weight is used by 128 or 256 rows per workgroup, so operands go through LDS (tile_mfma.hpp).
#include <algorithm>
#include <type_traits>
#include <vector>

#include "tile_mfma.hpp"

namespace salus {

// A wavefront's accumulators, whose first element is (m, n) of Y, to memory.  N is a multiple of 8, so a vector of 8
// (bf16) or 4 (float) columns lies wholly inside or outside.
template <int ACT, bool BF16, bool PAST_L2, int FN, int FM, typename Landed>
__device__ inline void store_dense(const Problem &p, uint32_t m, uint32_t n, const f32x16 (&acc)[FN][FM], int lane, Landed landed)
{
    constexpr int J = BF16 && FN % 2 == 0 ? 2 : 1;       // blocks that are stored together
    constexpr int kStores = BF16 ? 2 * J : 4, kRows = 32 / kStores;      // store instructions of them, rows of each
    const uint32_t N = p.N, esz = BF16 ? 2 : 4, pitch = N * esz;
    const uint32_t column = !BF16 ? line_column_f32(lane) : J == 2 ? line_column_bf16(lane) : half_line_column_bf16(lane);
    char *Y = (char *)p.Y + ((uint64_t)m * N + n) * esz;
    const char *aux = (const char *)p.aux + ((uint64_t)m * N + n) * 2;
    const bool mask = BF16 && (p.flags & kMaskPositive);
    const uint32_t rows = m < p.M ? p.M - m : 0, cols = n < N ? N - n : 0;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int j = 0; j < FN; j += J) {
            __builtin_amdgcn_sched_barrier(0);       // one line at a time: the accumulators leave few registers
            float v[J][16];
#pragma unroll
            for (int jj = 0; jj < J; ++jj)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float z = acc[j + jj][i][r];
                    v[jj][r] = ACT == 1 ? fmaxf(z, 0.0f) : ACT == 2 ? gelu_fast(z) : z;
                }
            __builtin_amdgcn_sched_barrier(0);
            if (i == 0 && j == 0) landed();
            const uint32_t c = 32u * j + column;
            u32x4 o[kStores];
            if constexpr (BF16 && J == 1) {
                to_half_lines_bf16(v[0], o);
            } else {
                std::conditional_t<BF16, u32x4, f32x4> lines[2][2];
                if constexpr (BF16) to_lines_bf16(v, lines);
                else to_lines_f32(v[0], lines);
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = __builtin_bit_cast(u32x4, lines[q >> 1][q & 1]);
            }
#pragma unroll
            for (int q = 0; q < kStores; ++q) {
                const uint32_t r_at = 32u * i + kRows * q + (lane & (kRows - 1));
                if (!(r_at < rows && c < cols)) continue;
                const uint32_t at = r_at * pitch + c * esz;
                u32x4 w = o[q];
                if (mask) {
                    // ReLU derivative taken from the stored bf16 activation (sign bit clear, not zero)
                    const u32x4 h = *(const u32x4 *)(aux + at);
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint32_t lo = h[d] & 0xffffu, hi = h[d] >> 16;
                        if ((lo & 0x8000u) || !lo) w[d] &= 0xffff0000u;
                        if ((hi & 0x8000u) || !hi) w[d] &= 0x0000ffffu;
                    }
                }
                if constexpr (PAST_L2) __builtin_nontemporal_store(w, (u32x4 *)(Y + at));
                else *(u32x4 *)(Y + at) = w;
            }
        }
    }
}

// Y = act(X . W) (TW: Y = X . W^T, W stored N x K, masked by the ReLU derivative)
template <int BM, int BN, bool TW>
struct DenseWalk {
    const GroupArgs &a;
    const uint32_t first;      // lane i: the first tile of problem i
    struct Place { int problem; uint32_t m0, n0, depth; };
    __device__ explicit DenseWalk(const GroupArgs &args) : a(args), first(args.first[threadIdx.x & 63]) {}
    __device__ uint32_t tiles() const { return a.tiles; }
    // Tiles of one job in bands of 8 row tiles, column tiles inside a band: the tiles an XCD runs at a time then share 8
    // slabs of X and 4 - 8 slabs of W in its L2.
    __device__ Place place(uint32_t tile_id) const
    {
        // the grid is a multiple of 8, so a workgroup's tiles all map to its own XCD's range
        const uint32_t id = xcd_remap(tile_id, a.tiles);
        const int g = __builtin_amdgcn_readfirstlane(wave_find_range(first, id, true));
        const Problem &p = a.p[g];
        const uint32_t t = id - __builtin_amdgcn_readlane(first, g), rt = (p.M + BM - 1) / BM, ct = (p.N + BN - 1) / BN;
        const uint32_t band = t / (8u * ct), local = t - band * 8u * ct, rows = min(8u, rt - band * 8u);
        return {g, (band * 8u + local % rows) * BM, (local / rows) * BN, p.K};
    }
    __device__ Operand m(const Place &at) const
    {
        const Problem &p = a.p[at.problem];
        return {p.X, p.K, p.M, p.K * 2u, false};
    }
    __device__ Operand n(const Place &at) const
    {
        const Problem &p = a.p[at.problem];
        if (TW) return {p.W, p.K, p.N, p.K * 2u, false};
        const bool strip = (p.flags & kStripW) != 0;
        return {p.W, p.K, p.N, strip ? 256u : p.N * 2u, strip};
    }
    struct Held {};            // nothing of the output is read
    __device__ void begin(const Place &, Held &, uint32_t, uint32_t, int) const {}
    template <int FN, int FM, typename Landed>
    __device__ void finish(const Place &at, const f32x16 (&acc)[FN][FM], const Held &, uint32_t m, uint32_t n, int lane, Landed landed) const
    {
        const Problem &p = a.p[at.problem];
        const uint32_t act = p.flags & 0xffu;
        m += at.m0;
        n += at.n0;
        auto store = [&](auto bf16, auto past_l2) {
            constexpr bool BF16 = decltype(bf16)::value, PAST = decltype(past_l2)::value;
            if (act == 1) store_dense<1, BF16, PAST>(p, m, n, acc, lane, landed);
            else if (act == 2) store_dense<2, BF16, PAST>(p, m, n, acc, lane, landed);
            else store_dense<0, BF16, PAST>(p, m, n, acc, lane, landed);
        };
        if (p.flags & kOutBf16) store(std::true_type{}, std::false_type{});
        else if (a.past_l2 && p.N % 32u == 0 && (uintptr_t)p.Y % 128u == 0) store(std::false_type{}, std::true_type{});
        else store(std::false_type{}, std::false_type{});
    }
};

// The workgroups are resident (one per compute unit, two of the 128 x 128 tile and of <128, 256, 1, 4>): workgroup b runs tiles b, b + grid, ...
// Bound, deep layers: the power limit.  16 jobs x 4096 rows, 4096 -> 1024: 480 us (1.14 PFLOP/s; 529 us with operands staged
// through registers and transposed on the way into LDS); 64 jobs: matrix pipes busy 65 % of the cycles at the 1.76 GHz that the
// chip then holds, no bank conflicts.  Layers of 16 slabs: the epilogue, which the one workgroup of a compute unit does with
// all its wavefronts at once, 128 outputs per lane (pipes 42 - 48 % at 1.9 GHz); under two workgroups per compute unit one multiplies
// meanwhile (32 jobs x 300 - 1000 rows, 1024 -> 4096: 46 % at 1.92 GHz).  1024 -> 4096 -> 1024 -> 1024 with GELU, 16 jobs x 4096 rows: 1180 - 1187 us (1421).
template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN, 2) void grouped_dense_bf16_tiled(GroupArgs a)
{
    using T = std::conditional_t<BM * BN == 128 * 256 && WM * WN == 4, TilePair<BM, BN, WM, WN>, TileMfma<BM, BN, WM, WN, false, true>>;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[T::kLds];
    const DenseWalk<BM, BN, false> walk(a);
    T::run(walk, smem);
}

// Two 128 x 256 tiles per compute unit for weights that come from HBM and that one row tile uses (jobs of up to 128 rows): bound by
// HBM, and asked for non-temporally they displace neither activations nor each other in L2.  64 jobs x 33 - 128 rows,
// 4096 -> 1024: 90 us (5.4 -> 6.0 TB/s of weights; 105 with plain requests), 1024 -> 4096 107 (115), the three layers of 1024 - 4096 -
// 1024 - 1024 246 (257); 39 jobs x 91 - 128 rows, 1288 -> 3576, rows of weights that begin inside a line, 99 (114).  Weights that the
// memory-side cache holds lose by it: 30 jobs x 65 - 128 rows, 1248 -> 2288: 45 plain, 58.
template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN, 2) void grouped_dense_bf16_tiled_once(GroupArgs a)
{
    using T = TilePair<BM, BN, WM, WN, true>;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[T::kLds];
    const DenseWalk<BM, BN, false> walk(a);
    T::run(walk, smem);
}

// WN x NS wavefronts share the columns.  Every wavefront of a 64 x 64 tile multiplies a 32 x 32 block through all of K:
// launches with at most one such tile per compute unit take 1.2 us less than with two wavefronts beside each other, the k-steps of a slab shared by
// two such groups and their sums added through LDS (10 jobs x 68 rows, 144 -> 656, 4.5 / 5.7 us; 5 jobs x 60 rows, 2664 -> 2912, 15.9 / 17.0).
// The order of its sums is that of those groups all the same: a wavefront keeps two, of the first and of the second half of every slab, and adds
// them at the end, half the length of a chain of roundings.  (InOrderArgs: one sum in order of k, as the 128 x 128 tiles that such launches
// took the place of have it.)
template <int BM, int BN, int WM, int WN, bool TW, int D, bool HALVES>
__device__ inline void stream_bf16(const GroupArgs &a)
{
    using T = TileStream<BM, BN, WM, WN, !TW, D, HALVES>;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[T::kLds];
    const DenseWalk<BM, BN, TW> walk(a);
    T::run(walk, smem);
}

template <int BM, int BN, int WM, int WN, int NS, bool TW, int D>
__global__ __launch_bounds__(64 * WM * WN * NS, WM * WN * NS / 2) void grouped_dense_bf16_stream(GroupArgs a)
{
    stream_bf16<BM, BN, WM, WN * NS, TW, D, BM * BN == 64 * 64>(a);
}
template <int BM, int BN, int WM, int WN, int NS, bool TW, int D>
__global__ __launch_bounds__(64 * WM * WN * NS, WM * WN * NS / 2) void grouped_dense_bf16_stream(InOrderArgs a)
{
    stream_bf16<BM, BN, WM, WN * NS, TW, D, false>(a);
}

bool tiled_shape_ok(const Problem &p) { return tiled_shape_fits(p) && p.K % kSlab == 0; }
// A depth that is no multiple of a slab costs the padding of the last slab, and one of up to four slabs leaves prologue and
// epilogue uncovered (below three there are whole slabs of zeros): such layers come here only if the round has enough
// of them (launch_grouped_bf16), ragged ones only from three slabs.
bool tiled_shape_ragged(const Problem &p)
{
    return tiled_shape_fits(p) && p.M > 128 && p.K % kSlab != 0 && p.K >= kMinSlabs * kSlab;
}
bool tiled_shape_shallow(const Problem &p) { return p.K <= 4 * kSlab; }
bool tiled_shape_fits(const Problem &p)
{
    return p.K != 0 && p.K % 8 == 0 && p.N % 8 == 0 && p.K < kTiledMaxWidth && p.N < kTiledMaxWidth;
}

uint64_t tiled_tiles(const Problem &p) { return (uint64_t)((p.M + 127) / 128) * ((p.N + 255) / 256); }

template <int BM, int BN, int PER_CU, typename Args = GroupArgs>
static hipError_t launch_tiled(void (*kernel)(Args), int threads, const Problem *p, uint32_t n, hipStream_t stream, uint64_t *launches)
{
    for (uint32_t at = 0; at < n; at += kMaxProblems) {
        Args a{};
        const uint64_t tiles = fill_group(a, p + at, std::min(kMaxProblems, n - at),
                                          [](const Problem &q) { return (uint64_t)((q.M + BM - 1) / BM) * ((q.N + BN - 1) / BN); });
        if (tiles == 0) continue;
        if (tiles > 0x7fffffffull) return hipErrorInvalidValue;
        // resident workgroups; a multiple of 8 so that the workgroups of an XCD keep to that XCD's range of tiles
        const uint32_t grid = (uint32_t)std::min<uint64_t>(tiles, resident_grid() * PER_CU);
        // Float outputs are a model's results, not read again here (a training step's logits are, without a difference): whole lines
        // of them go past L2 (non-temporal), as these stores bound wide shallow layers.  16 jobs x 4096 rows, 1024 -> 4096: 578 us, with plain stores 644; 32 jobs x 1000
        // rows, 256 -> 4096 131 / 174.  Not where rows do not begin on a line, whose pieces have to meet in L2 (256 -> 1000:
        // 68 / 38, see finish), nor with one workgroup per compute unit in one to three rounds, where its next tile waits for
        // the stores of the one before and nothing else covers that: 6 jobs x 1000 rows, 512 -> 4096, 1.09 of plain.  900
        // launches of 200 - 4096 rows: 6 % less on average.
        a.past_l2 = PER_CU == 2 || tiles < resident_grid() || tiles > 3 * (uint64_t)resident_grid();
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, stream, a);
        if (launches) *launches += 1;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Calibration: the multiply of a 256 x 256 tile without its memory
// traffic.  One workgroup of eight wavefronts per CU runs `slabs` times the 32
// MFMAs per wavefront of a 256 x 256 x 64 slab, either on fragments read once
// (lds == 0: what the matrix pipes sustain) or on fragments read from LDS for
// every k-step with one barrier per slab (lds != 0: the tiled kernel's multiply
// and LDS reads, nothing else).  Operands are nonzero (a pattern of small
// integers and fractions): the clock a matrix-bound kernel runs at depends on
// what the multipliers toggle.  Wavefront 0 of workgroup 0 reports the shader
// clocks and the 100 MHz ticks its loop took, so the clock under this load can
// be read off: out[0] = s_memtime difference, out[1] = wall-clock difference.
constexpr int kThreads2 = 512, kBK = 64, kBN = 256;
constexpr int kLine = kBK * 2;                 // bytes per LDS line
__device__ inline uint32_t swz(uint32_t line) { return (line ^ (line >> 3)) & 7u; }

template <bool LDS>
__global__ __launch_bounds__(kThreads2) void mfma_rate(uint64_t *out, uint32_t slabs)
{
    constexpr int BM = 256, FN = 4;
    __shared__ __attribute__((aligned(128))) unsigned char smem[2 * (BM + kBN) * kLine];
    for (uint32_t i = threadIdx.x; i < 2 * (BM + kBN) * kLine / 4; i += kThreads2) {
        const float a = 0.0625f * (float)((i * 7u) & 63u) - 2.0f, b = 0.03125f * (float)((i * 13u) & 127u) - 2.0f;
        ((uint32_t *)smem)[i] = bf16_pack(a, b);
    }
    __syncthreads();
    const uint32_t t = threadIdx.x, lane = t & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint32_t wm = wave >> 1, wn = wave & 1u;
    const uint32_t fl = lane & 31u, fh = lane >> 5, fs = swz(fl);
    const uint32_t afrag = (wm * 64u + fl) * kLine, bfrag = (BM + wn * 128u + fl) * kLine;
    f32x16 acc[2][FN];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    bf16x8 av[2], bv[FN];
    auto read = [&](const unsigned char *base, uint32_t ks) {
        const uint32_t off = ((2u * ks + fh) ^ fs) << 4, off_odd = off ^ 64u;
#pragma unroll
        for (int i = 0; i < 2; ++i) av[i] = *(const bf16x8 *)(base + afrag + 32 * i * kLine + (i & 1 ? off_odd : off));
#pragma unroll
        for (int j = 0; j < FN; ++j) bv[j] = *(const bf16x8 *)(base + bfrag + 32 * j * kLine + (j & 1 ? off_odd : off));
    };
    if (!LDS) read(smem, 0);
    const uint64_t c0 = __builtin_readcyclecounter(), w0 = wall_clock64();
    uint32_t stage = 0;
    for (uint32_t s = 0; s < slabs; ++s) {
#pragma unroll
        for (uint32_t ks = 0; ks < 4; ++ks) {
            if (LDS) read(smem + stage, ks);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        if (LDS) __syncthreads();
        stage ^= (BM + kBN) * kLine;
    }
    const uint64_t c1 = __builtin_readcyclecounter(), w1 = wall_clock64();
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += acc[i][j][r];
    if (blockIdx.x == 0 && t == 0) {
        out[0] = c1 - c0;
        out[1] = w1 - w0;
    }
    if (sum == 1.2345f) out[2] = 1;        // keeps the multiplies
}

// flop: what the launch computes (2 * 256 * 256 * 64 per slab and workgroup)
hipError_t launch_mfma_rate(uint64_t *dev_out, uint32_t slabs, bool lds, hipStream_t stream, uint64_t *flop)
{
    const uint32_t grid = resident_grid();
    if (lds) hipLaunchKernelGGL(mfma_rate<true>, dim3(grid), dim3(kThreads2), 0, stream, dev_out, slabs);
    else hipLaunchKernelGGL(mfma_rate<false>, dim3(grid), dim3(kThreads2), 0, stream, dev_out, slabs);
    if (flop) *flop = 2ull * 256 * 256 * 64 * slabs * grid;
    return hipGetLastError();
}

// Which tile a launch takes.  The grid walks its tiles in rounds of one (or two) per compute unit, so what counts is
// rounds x time of a round; a large tile moves fewer operand bytes per multiply but leaves the last round emptier
// and pads more.  Times of a round in nanoseconds, a slab and the rest (prologue and epilogue), fitted to launches of
// 16 jobs x 4096 rows, 4096 -> 1024 and 1024 -> 1024 (measured 480 / 161 us with 256 x 256 tiles, 536 / 175 with 128 x
// 256, 515 / 171 with two of those per compute unit, 612 / 201 with 128 x 128); of two tiles on a compute unit one ends
// while the other multiplies, so their rest counts less, and in a last round with at most one per compute unit a tile takes
// 0.6 of the time.  Two 128 x 256 tiles per compute unit also cover each other's waits for weights: where every weight
// is used by one row tile (up to 128 rows) and most compute units have one, half (64 jobs x 100 rows, 1024 -> 1024: 28 us,
// one per compute unit with twice the wavefronts 38; 24 jobs 20 / 18, so not there).  Over 528 launches of 33 - 4096 rows,
// 512 - 4096 -> 512 - 4096, the choice is 1.0 % off the best kind on average; without that kind it was 2.4 % slower.  Weights from HBM cost
// one round of 256 x 256 tiles, which ask for every weight once per 256 rows, less than what the others need more rounds for: 5 jobs x
// 500 rows, 1280 -> 3968, 256 x 256 / 128 x 128 37.8 / 37.0 us from the cache, 38.3 / 47.6 from HBM; 18 jobs x 256 - 1024, 1024 -> 896, 30.4 / 29.1 and
// 32.9 / 38.6.  7 % off its time then (any figure from there to 20 % gives the same choices but one): over 207 launches of 65 - 1024 rows with weights from
// HBM the choice is 1.4 % off the best kind, 2.0 % without; and 7 % off that of two 128 x 256 tiles that ask for weights
// non-temporally (grouped_dense_bf16_tiled_once, 3 - 12 % less than with plain requests) where most compute units have one (10 jobs x 33 - 67 rows, 1792 -> 3456,
// 140 tiles, 36.4 / 26.9 us of one per compute unit with twice the wavefronts) and rows of an operand begin inside a line, which 128 x 128 tiles
// ask for more pieces of: of 19 such launches whose choice that changes, 128 x 128 / once, 46 jobs x 49 - 110 rows, 2344 -> 3072, 181 / 152 us, 63 jobs x 72 -
// 113, 1616 -> 1168, 76.8 / 70.8, 0.94 on average and never more than 1.00.  Whole lines keep the times as they are: 55 jobs x 96 - 126, 1024 -> 1280, 44.9 / 47.3,
// 23 jobs x 93 - 128, 768 -> 3072, 36.7 / 39.4, 57 jobs x 53 - 101, 2944 -> 1280, 99.2 / 102.4, 1.007 on average over 25; what stays slower for it: 52 jobs x 38 -
// 71, 2432 -> 3072, 150.7 / 146.7, 46 jobs x 75, 1536 -> 3328, 98.0 / 96.4.  What the rule is
// for: 4 jobs x 500 rows, 2048 -> 2048, 256 x 256 / 128 x 256 / 128 x 128 / two 128 x 256: 48 / 30 / 25 / 33 us; 32 jobs x
// 300 - 1000 rows, 4096 -> 1024 207 / 200 / 222 / 195, 1024 -> 1024 70 / 69 / 61 / 55; 32 jobs x 500 rows, 1024 -> 4096 167 /
// 190 / 222 / 181.
struct TileKind { uint32_t bm, bn, per_cu, slab_ns, rest_ns; };
constexpr TileKind kTile256 = {256, 256, 1, 1640, 12000}, kTile128x256 = {128, 256, 1, 935, 8000}, kTile128 = {128, 128, 2, 1090, 6000},
                   kTilePair = {128, 256, 2, 1720, 12000};

static uint64_t launch_ns(const TileKind &t, const Problem *p, uint32_t n, bool cached)
{
    uint64_t tiles = 0, work = 0;
    bool weight_bound = true, lines = true;
    for (uint32_t i = 0; i < n; ++i) {
        const uint64_t count = (uint64_t)((p[i].M + t.bm - 1) / t.bm) * ((p[i].N + t.bn - 1) / t.bn);
        tiles += count;
        work += count * (((uint64_t)p[i].K + kSlab - 1) / kSlab * t.slab_ns + t.rest_ns);
        weight_bound = weight_bound && p[i].M <= 128;
        lines = lines && p[i].K % 64 == 0 && ((p[i].flags & kStripW) || p[i].N % 64 == 0);
    }
    if (tiles == 0) return 0;
    const uint64_t cus = resident_grid(), grid = cus * t.per_cu, last = tiles % grid;
    uint64_t tenths = tiles / grid * 10;       // of a round
    if (last) tenths += t.per_cu == 1 || last > cus ? 10 : &t == &kTilePair && weight_bound && last * 4 > cus * 3 ? 5 : 6;
    const uint64_t ns = tenths * (work / tiles) / 10;
    const bool less = &t == &kTile256 ? tiles <= cus : &t == &kTilePair && weight_bound && !lines && tiles * 4 > cus * 3;
    return !cached && less ? ns * 93 / 100 : ns;
}

// What the launch of two 128 x 256 tiles per compute unit asks for non-temporally.
static bool weights_once(const Problem *p, uint32_t n, bool cached)
{
    return !cached && std::all_of(p, p + n, [](const Problem &q) { return q.M <= 128; });
}

// Launches bound by the weight stream.  64 x 128 tiles, two workgroups per compute unit; 64 x 64, twice the workgroups,
// while there is at most one of them per compute unit (transposed weights: while 64 x 128 would be fewer than one).  64 x
// 128 / 64 x 64: 12 jobs x 64 rows, 2048 -> 1536 26 / 33 us, 20 jobs x 33 - 128 rows, 4096 -> 1024 47 / 56, 16 jobs x 33 -
// 100 rows, 1536 -> 768 19 / 21, 8 jobs x 64 rows, 2048 -> 2048 with weights from memory 27 / 22.5; 8 jobs x 100 rows: 64 x 128 tiles, training
// step 386 us against 410 with 64 x 64 (all of these with the k-steps of a 64 x 64 tile shared by two groups of wavefronts).  While
// there is at most one 64 x 128 tile per compute unit, eight wavefronts instead of four for jobs of 128 rows and more, four / eight: 3 jobs x 300 rows, 2048 -> 1536,
// 16.4 / 15.1 us, 4 jobs x 200, 4096 -> 1536, 29.7 / 28.1, 7 jobs x 234, 1088 -> 728, 10.5 / 9.9, 5 jobs x 200, 2120 -> 1288, 17.9 / 17.3; from HBM the same within 3 %
// (16 jobs x 128 rows, 1024 -> 1024, 15.6 / 16.0), and beyond one tile as well.  Not for one row tile whose weights come from HBM (10 jobs x 33 - 60 rows, 1992 -> 2536, 26.4 / 27.3).
// Jobs of 65 - 127 rows, which have two row tiles too, keep four: eight are 3 - 8 % quicker there from the cache (nine launches; 7 jobs x 127 rows, 1536 -> 2048, 14.2 /
// 13.2) and as quick from HBM, so the line could lie at 65.  Rings of six and eight
// slabs for one 64 x 64 tile per compute unit: step of 8 jobs x 64 rows 313 and 317 us, with four 301.
hipError_t launch_grouped_bf16_stream(const Problem *p, uint32_t n, bool trans_w, bool in_order, hipStream_t stream, uint64_t *launches)
{
    uint64_t wide = 0, narrow = 0;
    for (uint32_t i = 0; i < n; ++i) {
        if (!tiled_shape_fits(p[i])) return hipErrorInvalidValue;
        wide += (uint64_t)((p[i].M + 63) / 64) * ((p[i].N + 127) / 128);
        narrow += (uint64_t)((p[i].M + 63) / 64) * ((p[i].N + 63) / 64);
    }
    const bool few = trans_w ? wide < resident_grid() : narrow <= resident_grid();
    if (few && trans_w) return launch_tiled<64, 64, 2>(grouped_dense_bf16_stream<64, 64, 2, 1, 2, true, 4>, 256, p, n, stream, launches);
    if (few && in_order) return launch_tiled<64, 64, 2, InOrderArgs>(grouped_dense_bf16_stream<64, 64, 2, 1, 2, false, 4>, 256, p, n, stream, launches);
    if (few) return launch_tiled<64, 64, 2>(grouped_dense_bf16_stream<64, 64, 2, 1, 2, false, 4>, 256, p, n, stream, launches);
    if (trans_w) return launch_tiled<64, 128, 2>(grouped_dense_bf16_stream<64, 128, 2, 2, 1, true, 3>, 256, p, n, stream, launches);
    if (wide <= resident_grid() && std::all_of(p, p + n, [](const Problem &q) { return q.M >= 128; }))
        return launch_tiled<64, 128, 2>(grouped_dense_bf16_stream<64, 128, 2, 2, 2, false, 3>, 512, p, n, stream, launches);
    return launch_tiled<64, 128, 2>(grouped_dense_bf16_stream<64, 128, 2, 2, 1, false, 3>, 256, p, n, stream, launches);
}

// The tile for these jobs (256 rows only if all have the rows for it) and the time it takes.  Shallow layers are all
// epilogue, which only two tiles on a compute unit overlap: 128 x 128 (160 launches of 256 -> 1024 and 4096, 192 - 4096 rows:
// 1 % off the best kind on average, 128 x 256 11 %, 256 x 256 28 %).
struct TileChoice { const TileKind *kind; uint64_t ns; };
static TileChoice choose_tile(const std::vector<Problem> &p, bool tall, bool cached)
{
    TileChoice best{nullptr, ~0ull};
    if (p.empty()) return best;
    const bool shallow = std::all_of(p.begin(), p.end(), tiled_shape_shallow);
    for (const TileKind *t : {&kTile256, &kTile128x256, &kTile128, &kTilePair}) {
        if ((t == &kTile256 && !tall) || (t != &kTile128 && shallow)) continue;
        const uint64_t ns = launch_ns(*t, p.data(), (uint32_t)p.size(), cached);
        if (ns < best.ns) best = {t, ns};
    }
    return best;
}

hipError_t launch_grouped_bf16_tiled(const Problem *p, uint32_t n, bool cached, hipStream_t stream, uint64_t *launches)
{
    std::vector<Problem> big, small;
    bool ragged = false;
    for (uint32_t i = 0; i < n; ++i) {
        if (!tiled_shape_fits(p[i])) return hipErrorInvalidValue;
        ragged = ragged || tiled_shape_ragged(p[i]);
    }
    big.reserve(n);
    for (uint32_t i = 0; i < n; ++i) (p[i].M >= kTiled256MinM ? big : small).push_back(p[i]);
    TileChoice tall = choose_tile(big, true, cached);
    const TileChoice low = choose_tile(small, false, cached);
    if (ragged && !big.empty() && !small.empty()) {
        // Jobs on either side of 192 rows, ragged ones among them (whose alternative, register tiles, is one launch): one
        // launch of 128-row tiles, unless two are quicker even though each ends with a round of its own.  16 jobs x
        // 129 - 260 rows, 2056 -> 520: 21 us, in two launches 42.
        const std::vector<Problem> all(p, p + n);
        const TileChoice one = choose_tile(all, false, cached);
        if (one.ns <= tall.ns + low.ns) {
            big = all;
            small.clear();
            tall = one;
        }
    }
    for (const std::vector<Problem> *group : {&big, &small}) {
        if (group->empty()) continue;
        const Problem *q = group->data();
        const uint32_t count = (uint32_t)group->size();
        const TileKind *kind = group == &big ? tall.kind : low.kind;
        const hipError_t e = kind == &kTile256       ? launch_tiled<256, 256, 1>(grouped_dense_bf16_tiled<256, 256, 2, 4>, 512, q, count, stream, launches)
                             : kind == &kTilePair    ? launch_tiled<128, 256, 2>(weights_once(q, count, cached) ? grouped_dense_bf16_tiled_once<128, 256, 1, 4> : grouped_dense_bf16_tiled<128, 256, 1, 4>,
                                                                                 256, q, count, stream, launches)
                             : kind == &kTile128x256 ? launch_tiled<128, 256, 1>(grouped_dense_bf16_tiled<128, 256, 2, 4>, 512, q, count, stream, launches)
                                                     : launch_tiled<128, 128, 2>(grouped_dense_bf16_tiled<128, 128, 2, 2>, 256, q, count, stream, launches);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace salus
