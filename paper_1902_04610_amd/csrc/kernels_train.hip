// Training-step kernels for gfx950: softmax cross-entropy with its gradient,
// and the fused weight-gradient + SGD update.  (The input-gradient product
// dX = dY . W^T reuses grouped_dense_bf16 with the transposed-weight load path.)
//
// A training iteration is a forward pass, a backward pass and a parameter
// update (Salus paper, Section 2.1); hyper-parameter tuning packs many such
// jobs of one architecture on a GPU (Section 5.2).  All jobs of a round share
// every launch here, as in the forward pass.
#include <algorithm>

#include "tile_mfma.hpp"

namespace salus {

__device__ inline uint32_t bf16_rne(float f) { return bf16_bits(f); }

__device__ inline float wave_max(float v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
}

__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// ---------------------------------------------------------------------------
// Mean softmax cross-entropy over the M rows of each job and its gradient
// (softmax - onehot) / M, written as bf16 for the backward products.  A
// workgroup of 16 wavefronts takes 16 rows of one job (the job is found with the
// lookup used everywhere else), one wavefront one row: the rows are spread over as many
// compute units as there are, since one unit's memory path is what bounds it (8 jobs x 64 rows x 1000 classes:
// 5.3 us, with 64 rows per workgroup 13 us).  Rows of up to
// 1024 classes are read once and kept in registers; wider rows are re-read from memory for each of the three
// passes.  Row losses are added in row order, so the result does
// not depend on how the rows were scheduled: inside the workgroup when it holds
// the whole job, else over the scratch array, by the launch that updates the weights or, where the scratch
// array cannot live that long, by a second, tiny kernel (5 us of a step).
// ---------------------------------------------------------------------------
struct LossArgs {
    uint32_t n;
    uint32_t tiles;      // blocks of kLossRows rows
    uint32_t first[kMaxProblems];      // first block of job i; kNoTile from n on
    LossProblem p[kMaxProblems];
};

constexpr int kLossWaves = 16, kLossPerWave = kLossRows / kLossWaves, kLossRegs = 16;

__global__ __launch_bounds__(64 * kLossWaves) void softmax_xent_rows(LossArgs a)
{
    __shared__ float row_loss[kLossRows];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    LossProblem p;
    const uint32_t row0 = find_owner(a.first, a.p, blockIdx.x, p) * kLossRows;
    const uint32_t M = p.M, N = p.N;
    const Global<float> *logits = (const Global<float> *)p.logits;
    Global<float> *row_losses = (Global<float> *)p.row_loss;
    const float inv_m = 1.0f / (float)M;
    // register path: lane owns classes 256 i + 4 lane .. + 3 of a row (16-byte loads, 8-byte stores)
    const bool in_regs = N <= 64u * kLossRegs && N % 4 == 0;

    f32x4 zr[kLossPerWave][kLossRegs / 4];
    int labels[kLossPerWave];
#pragma unroll
    for (int q = 0; q < kLossPerWave; ++q) {
        const uint32_t row = row0 + wave * kLossPerWave + q;
        const int l = ((const Global<int32_t> *)p.labels)[row < M ? row : M - 1];
        labels[q] = l < 0 ? 0 : (l >= (int)N ? (int)N - 1 : l);          // never read outside the row
    }
    if (in_regs) {
#pragma unroll
        for (int q = 0; q < kLossPerWave; ++q) {
            const uint32_t row = row0 + wave * kLossPerWave + q;
            const Global<float> *z = logits + (size_t)(row < M ? row : M - 1) * N;
#pragma unroll
            for (int i = 0; i < kLossRegs / 4; ++i) {
                const uint32_t n = 256u * i + 4u * lane;
                zr[q][i] = *(const Global<f32x4> *)(z + (n < N ? n : N - 4));
            }
        }
    }
#pragma unroll
    for (int q = 0; q < kLossPerWave; ++q) {
        const uint32_t row = row0 + wave * kLossPerWave + q;
        if (row >= M) continue;                              // uniform per wavefront
        const Global<float> *z = logits + (size_t)row * N;
        Global<uint16_t> *g = (Global<uint16_t> *)p.grad + (size_t)row * N;
        const int label = labels[q];
        float zmax = -INFINITY, denom = 0.0f, zlabel = 0.0f;
        if (in_regs) {
#pragma unroll
            for (int i = 0; i < kLossRegs / 4; ++i)
                if (256u * i + 4u * lane < N)
                    zmax = fmaxf(fmaxf(zmax, fmaxf(zr[q][i][0], zr[q][i][1])), fmaxf(zr[q][i][2], zr[q][i][3]));
            zmax = wave_max(zmax);
            f32x4 e[kLossRegs / 4];
#pragma unroll
            for (int i = 0; i < kLossRegs / 4; ++i) {
                // v_exp_f32: error at the last-bit level, far below the bf16 rounding of the gradient
#pragma unroll
                for (int j = 0; j < 4; ++j) e[i][j] = __expf(zr[q][i][j] - zmax);
                if (256u * i + 4u * lane < N) denom += (e[i][0] + e[i][1]) + (e[i][2] + e[i][3]);
            }
            denom = wave_sum(denom);
            const float inv_d = 1.0f / denom;
#pragma unroll
            for (int i = 0; i < kLossRegs / 4; ++i) {
                const uint32_t n = 256u * i + 4u * lane;
                if (n >= N) continue;
                float h[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool hit = (int)(n + j) == label;
                    if (hit) zlabel = zr[q][i][j];
                    h[j] = (e[i][j] * inv_d - (hit ? 1.0f : 0.0f)) * inv_m;
                }
                *(Global<u32x2> *)(g + n) = u32x2{bf16_pack(h[0], h[1]), bf16_pack(h[2], h[3])};
            }
            // the lane that holds the label's class hands its logit to lane 0
            zlabel = __shfl(zlabel, (label & 255) >> 2, 64);
        } else {
            for (uint32_t n = lane; n < N; n += 64) zmax = fmaxf(zmax, z[n]);
            zmax = wave_max(zmax);
            for (uint32_t n = lane; n < N; n += 64) denom += expf(z[n] - zmax);
            denom = wave_sum(denom);
            const float inv_d = 1.0f / denom;
            for (uint32_t n = lane; n < N; n += 64) {
                const float prob = expf(z[n] - zmax) * inv_d;
                g[n] = (uint16_t)bf16_rne((prob - ((int)n == label ? 1.0f : 0.0f)) * inv_m);
            }
        }
        if (!in_regs) zlabel = z[label];
        if (lane == 0) {
            const float loss = -(zlabel - zmax - logf(denom));
            row_loss[row - row0] = loss;
            if (M > kLossRows) row_losses[row] = loss;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && M <= kLossRows) {      // this workgroup holds the whole job
        float sum = 0.0f;
#pragma unroll
        for (uint32_t r = 0; r < kLossRows; ++r) {
            const float v = row_loss[r < M ? r : 0];
            if (r < M) sum += v;
        }
        *(Global<float> *)p.loss = sum / (float)M;
    }
}

// Jobs of more than 16 rows, one wavefront: add the row losses of one in row order: 512 of them are loaded at a time and added lane by
// lane (500 rows: 5 us; a load per row took 23 us).
__device__ inline void mean_of_rows(const float *row_loss, uint32_t M, float *loss)
{
    const uint32_t lane = threadIdx.x & 63;
    float sum = 0.0f;
    for (uint32_t r0 = 0; r0 < M; r0 += 512) {
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint32_t r = r0 + 64u * c + lane;
            v[c] = r < M ? ((const Global<float> *)row_loss)[r] : 0.0f;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (r0 + 64u * c >= M) break;
#pragma unroll
            for (int i = 0; i < 64; ++i) sum += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v[c]), i));
        }
    }
    if (lane == 0) *(Global<float> *)loss = sum / (float)M;
}

__global__ __launch_bounds__(64) void loss_mean(LossArgs a)
{
    const LossProblem &p = a.p[blockIdx.x];
    if (p.M > kLossRows) mean_of_rows(p.row_loss, p.M, p.loss);
}

hipError_t launch_softmax_xent(const LossProblem *p, uint32_t n, bool mean_later, hipStream_t stream, uint64_t *launches)
{
    for (uint32_t at = 0; at < n; at += kMaxProblems) {
        LossArgs a{};
        const uint32_t count = std::min(kMaxProblems, n - at);
        const uint64_t blocks = fill_group(a, p + at, count, [](const LossProblem &q) { return (uint64_t)((q.M + kLossRows - 1) / kLossRows); });
        const bool big = std::any_of(p + at, p + at + count, [](const LossProblem &q) { return q.M > kLossRows; });
        if (blocks == 0) continue;
        if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
        hipLaunchKernelGGL(softmax_xent_rows, dim3((uint32_t)blocks), dim3(64 * kLossWaves), 0, stream, a);
        if (big && !mean_later) hipLaunchKernelGGL(loss_mean, dim3(a.n), dim3(64), 0, stream, a);
        if (launches) *launches += 1;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// dW = H^T . G fused with the SGD update.  The contraction runs over the batch
// (M rows, 32 per MFMA step), so per weight there are only M multiply-adds and
// the kernel is bound by the read-modify-write of the float master weights
// (4 B read, 4 B + 2 B written per weight).
//
// One wavefront owns a KB (k) x 64 (n) block of W, KB = 16 KI; a workgroup is four such
// blocks side by side.  Lane (c, g) loads the 8 x KI blocks H[m0+8g ..][k0+KI*c ..]
// and 8 x 4 blocks G[m0+8g ..][n0+4c ..], transposes them in registers into
// KI A and four B operands of v_mfma_f32_16x16x32_bf16; MFMA (i, j) yields
// rows k0 + KI*rho + i, columns n0 + 4*c + j.  A lane ends up with 4 KI rows x 4
// consecutive columns, so master weights move as 16-byte vectors, 256
// contiguous bytes per row across the 16 lanes.
// ---------------------------------------------------------------------------
struct UpdateArgs {
    uint32_t n;
    uint32_t tiles;      // all tiles of the launch
    uint32_t losses;     // n if a mean loss is to be taken, else 0
    uint32_t first[kMaxProblems];      // first tile of update i; kNoTile from n on
    UpdateProblem p[kMaxProblems];
    float *loss[kMaxProblems];
};
static_assert(sizeof(UpdateArgs) <= 4096, "kernel arguments are limited to 4 KB");

constexpr int kUpdK = 64, kUpdFewK = 32, kUpdN = 256;      // workgroup tiles
constexpr int kUpdSteps = 4;                // steps of 32 rows that a tile of few rows requests at once
constexpr double kDwTiledRows = 192;
constexpr int kDwTile = 128;                // tile of the many-row kernel

// The mean loss that belongs to update `i` of the launch, if one does: a workgroup's first wavefront's work beside its tile.  Behind it, if that is the only
// one: in front the look for a loss alone was 0.25 us of a launch of few blocks (6.1 us), also where no job has one.
__device__ inline void dw_mean_loss(const UpdateArgs &a, uint32_t i)
{
    if (i >= a.losses || threadIdx.x >= 64) return;
    const UpdateProblem &p = a.p[i];
    if (a.loss[i]) mean_of_rows((const float *)((const uint16_t *)p.G + (size_t)p.M * p.N), p.M, a.loss[i]);
}

template <typename Tiles>
static uint64_t fill_updates(UpdateArgs &a, const UpdateWithLoss *p, uint32_t n, Tiles tiles)
{
    for (uint32_t i = 0; i < n; ++i) {
        a.loss[i] = p[i].loss;
        if (p[i].loss) a.losses = n;
    }
    return fill_group(a, p, n, tiles);
}

// One step of 32 rows: a lane's blocks h and d into operands, and their products.
template <int KI, typename HVec>
__device__ inline void dw_multiply(const HVec (&h)[8], const u32x2 (&d)[8], f32x4 (&acc)[4 * KI])
{
    u32x4 A[KI], B[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;
            if (i < KI) A[i][j] = __builtin_amdgcn_perm(h[2 * j + 1][i >> 1], h[2 * j][i >> 1], sel);
            B[i][j] = __builtin_amdgcn_perm(d[2 * j + 1][i >> 1], d[2 * j][i >> 1], sel);
        }
#pragma unroll
    for (int i = 0; i < KI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i * 4 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, A[i]), __builtin_bit_cast(bf16x8, B[j]), acc[i * 4 + j],
                0, 0, 0);
}

// Master weights of a lane: rows first + KI * r + i, columns ncol .. ncol+3.
template <int KI>
__device__ inline void dw_load(const UpdateProblem &p, uint32_t first, uint32_t ncol, f32x4 (&wm)[4 * KI])
{
    const Global<float> *Wm = (const Global<float> *)p.Wm;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < KI; ++i) {
            const uint32_t krow = first + KI * r + i;
            wm[r * KI + i] = (krow < p.K && ncol < p.N)
                                 ? __builtin_nontemporal_load((const Global<f32x4> *)(Wm + (size_t)krow * p.N + ncol))
                                 : f32x4{0.f, 0.f, 0.f, 0.f};
        }
}

template <int KI>
__device__ inline void dw_store(const UpdateProblem &p, uint32_t first, uint32_t ncol, const f32x4 (&wm)[4 * KI], const f32x4 (&acc)[4 * KI])
{
    Global<float> *Wm = (Global<float> *)p.Wm;
    Global<uint16_t> *Wb = (Global<uint16_t> *)p.Wb;
    const float lr = p.lr;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < KI; ++i) {
            const uint32_t krow = first + KI * r + i;
            if (krow >= p.K || ncol >= p.N) continue;
            f32x4 w = wm[r * KI + i];
#pragma unroll
            for (int j = 0; j < 4; ++j)      // one rounded multiply, one rounded subtract
                w[j] = __fsub_rn(w[j], __fmul_rn(lr, acc[i * 4 + j][r]));
            __builtin_nontemporal_store(w, (Global<f32x4> *)(Wm + (size_t)krow * p.N + ncol));
            u32x2 b;
            b[0] = bf16_pack(w[0], w[1]);
            b[1] = bf16_pack(w[2], w[3]);
            *(Global<u32x2> *)(Wb + (size_t)krow * p.N + ncol) = b;
        }
}

// Blocks of 64 x 64.  The master-weight loads are issued before the MFMA phase and complete underneath it.
__global__ __launch_bounds__(256) void grouped_dw_sgd(UpdateArgs a)
{
    UpdateProblem p;
    const uint32_t t = find_owner(a.first, a.p, blockIdx.x, p);
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t M = p.M, K = p.K, N = p.N, kt = (K + kUpdK - 1) / kUpdK;
    const uint32_t k0 = (t % kt) * kUpdK;                  // neighbours share the G columns
    const uint32_t n0 = (t / kt) * kUpdN + 64 * wave;
    const uint32_t ncol = n0 + 4 * c;
    const bool col_ok = ncol < N;
    const Global<uint16_t> *H = (const Global<uint16_t> *)p.H;
    const Global<uint16_t> *G = (const Global<uint16_t> *)p.G;
    f32x4 wm[16], acc[16];      // acc[i * 4 + j][r]
    dw_load<4>(p, k0 + 16 * g, ncol, wm);
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t kcol = k0 + 4 * c;
    const bool kcol_ok = kcol < K;
    for (uint32_t m0 = 0; m0 < M; m0 += 32) {
        u32x2 h[8], d[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const uint32_t m = m0 + 8 * g + r;
            h[r] = (m < M && kcol_ok) ? *(const Global<u32x2> *)(H + (size_t)m * K + kcol) : u32x2{0u, 0u};
            d[r] = (m < M && col_ok) ? *(const Global<u32x2> *)(G + (size_t)m * N + ncol) : u32x2{0u, 0u};
        }
        dw_multiply<4>(h, d, acc);
    }
    dw_store<4>(p, k0 + 16 * g, ncol, wm, acc);
    dw_mean_loss(a, blockIdx.x);
}

// Few rows: blocks of 32 x 64.  What a block waits for is requested at once, up to 128 rows of H and G and behind them its master weights, which
// arrive under the multiplies: a block that asks for 32 rows at a time waits behind HBM's queue with each of them.  The registers that
// takes leave two workgroups per compute unit, which is no loss (three, with 64 rows at once, are slower).  Tiles of a row of
// blocks are neighbours, so that what is under way at a time is whole rows of W.  More rows take blocks of 64 x 64, which
// ask L2 for H and G two thirds as often (launch_grouped_dw_sgd).
// 8 jobs x 64 rows, 2048 - 2048 - 2048 - 2048 - 1000 (1.17 GB), kernel trace of twenty steps: 196 us (192 - 201), blocks of 64 x 64 205 (199 - 210), on
// another card 200 - 205 and 210 - 212; 8 rows 172 / 184.  (55 steps of bench.py: 194 on average, 188 - 203.)
__global__ __launch_bounds__(256, 2) void grouped_dw_sgd_few_rows(UpdateArgs a)
{
    UpdateProblem p;
    const uint32_t t = find_owner(a.first, a.p, blockIdx.x, p);
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t M = p.M, K = p.K, N = p.N, nt = (N + kUpdN - 1) / kUpdN;
    // Workgroups go round-robin to 8 XCDs.  Where a row of blocks ends with a partial one, which would recur on the same XCDs (8 blocks: always on the last),
    // rows are turned: steps of 4 jobs x 64 rows of 1192 - 1832 - 824 - 1840 - 360 121.6 us (125.2), of 784 - 1592 - 312 48.4 (50.4).  Not where it is nearly
    // whole: a column of blocks that keeps to its XCD finds its part of G in that L2 (8 jobs, 2048 wide: 323.8 us turned, 316.5).
    const uint32_t row = t / nt, turn = N % kUpdN - 1u < 192u ? row * min(nt & -nt, 8u) / 8 : 0u;
    const uint32_t k0 = row * kUpdFewK, n0 = (t + turn) % nt * kUpdN + 64 * wave;
    const uint32_t ncol = n0 + 4 * c, kcol = k0 + 2 * c;
    const bool col_ok = ncol < N;
    // rows and columns outside the matrices: a valid address, and what comes of it is not stored
    const Global<uint16_t> *H = (const Global<uint16_t> *)p.H + (kcol < K ? kcol : 0);
    const Global<uint16_t> *G = (const Global<uint16_t> *)p.G + (col_ok ? ncol : 0);
    f32x4 acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    typedef unsigned int u32x1 __attribute__((ext_vector_type(1)));
    u32x1 h[kUpdSteps][8];
    u32x2 d[kUpdSteps][8];
    auto load = [&](int s, uint32_t m0) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const size_t m = min(m0 + 8 * g + r, M - 1);
            h[s][r] = *(const Global<u32x1> *)(H + m * K);
            d[s][r] = *(const Global<u32x2> *)(G + m * N);
        }
    };
    auto multiply = [&](int s, uint32_t m0) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (m0 + 8 * g + r >= M) {
                h[s][r] = u32x1{0u};
                d[s][r] = u32x2{0u, 0u};
            }
        dw_multiply<2>(h[s], d[s], acc);
    };
#pragma unroll
    for (int s = 0; s < kUpdSteps; ++s)
        if (32u * s < M) load(s, 32u * s);
    __builtin_amdgcn_sched_barrier(0);
    f32x4 wm[8];
    dw_load<2>(p, k0 + 8 * g, ncol, wm);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < kUpdSteps; ++s)
        if (32u * s < M) multiply(s, 32u * s);
    for (uint32_t m0 = 32 * kUpdSteps; m0 < M; m0 += 32 * kUpdSteps) {
#pragma unroll
        for (int s = 0; s < kUpdSteps; ++s)
            if (m0 + 32u * s < M) load(s, m0 + 32u * s);
#pragma unroll
        for (int s = 0; s < kUpdSteps; ++s)
            if (m0 + 32u * s < M) multiply(s, m0 + 32u * s);
    }
    dw_store<2>(p, k0 + 8 * g, ncol, wm, acc);
    dw_mean_loss(a, blockIdx.x);
}

// Many rows per job (the contraction is long): the product goes through the LDS tiles of tile_mfma.hpp, both operands
// transposed on the way out of LDS.  M side: H (rows of W), N side: G (columns of W).
struct UpdateWalk {
    const UpdateArgs &a;
    const uint32_t first;      // lane i: the first tile of update i
    struct Place { int problem; uint32_t m0, n0, depth; };
    __device__ explicit UpdateWalk(const UpdateArgs &args) : a(args), first(args.first[threadIdx.x & 63]) {}
    __device__ uint32_t tiles() const { return a.tiles; }
    // Columns first: the tiles under way at a time touch whole rows of the master weights (8 jobs x 256 rows: 454 us a step, rows
    // first 470).
    __device__ Place place(uint32_t tile_id) const
    {
        const uint32_t id = xcd_remap(tile_id, a.tiles);
        const int g = __builtin_amdgcn_readfirstlane(wave_find_range(first, id, true));
        const uint32_t t = id - __builtin_amdgcn_readlane(first, g), nt = (a.p[g].N + kDwTile - 1) / kDwTile;
        return {g, (t / nt) * kDwTile, (t % nt) * kDwTile, a.p[g].M};
    }
    __device__ Operand m(const Place &at) const { const UpdateProblem &p = a.p[at.problem]; return {p.H, p.M, p.K, p.K * 2u, false}; }
    __device__ Operand n(const Place &at) const { const UpdateProblem &p = a.p[at.problem]; return {p.G, p.M, p.N, p.N * 2u, false}; }
    // The master weights of a wavefront's part of a tile, requested in front of its multiplies: the second slab waits for them
    // (loads complete in order), the update does not.
    static constexpr int kF = kDwTile / 2 / 32;      // blocks of 32 rows or columns in it
    struct Held { f32x4 w[kF][kF][2][2]; };
    struct Part { float *Wm; uint16_t *Wb; uint32_t N, rows, cols; };
    __device__ Part part(const Place &at, uint32_t m, uint32_t n) const
    {
        const UpdateProblem &p = a.p[at.problem];
        m += at.m0;
        n += at.n0;
        const uint64_t corner = (uint64_t)m * p.N + n;
        return {p.Wm + corner, (uint16_t *)p.Wb + corner, p.N, m < p.K ? p.K - m : 0, n < p.N ? p.N - n : 0};
    }
    __device__ void begin(const Place &at, Held &held, uint32_t m, uint32_t n, int lane) const
    {
        const Part p = part(at, m, n);
        const uint32_t column = line_column_f32(lane);
#pragma unroll
        for (int i = 0; i < kF; ++i)
#pragma unroll
            for (int j = 0; j < kF; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t r = 32u * i + 8u * q + (lane & 7), c = 32u * j + column;
                    held.w[j][i][q >> 1][q & 1] = r < p.rows && c < p.cols ? __builtin_nontemporal_load((const f32x4 *)(p.Wm + (size_t)r * p.N + c))
                                                                           : f32x4{0.f, 0.f, 0.f, 0.f};
                }
    }
    template <int FN, int FM, typename Landed>
    __device__ void finish(const Place &at, const f32x16 (&acc)[FN][FM], const Held &held, uint32_t m, uint32_t n, int lane, Landed landed) const
    {
        const Part p = part(at, m, n);
        const uint32_t N = p.N, rows = p.rows, cols = p.cols, column = line_column_f32(lane);
        float *Wm = p.Wm;
        uint16_t *Wb = p.Wb;
        const float lr = a.p[at.problem].lr;
        landed();
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                float v[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = acc[j][i][r];
                f32x4 o[2][2];
                to_lines_f32(v, o);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t r = 32u * i + 8u * q + (lane & 7), c = 32u * j + column;
                    if (!(r < rows && c < cols)) continue;
                    f32x4 x = held.w[j][i][q >> 1][q & 1];
#pragma unroll
                    for (int e = 0; e < 4; ++e)      // one rounded multiply, one rounded subtract
                        x[e] = __fsub_rn(x[e], __fmul_rn(lr, o[q >> 1][q & 1][e]));
                    __builtin_nontemporal_store(x, (f32x4 *)(Wm + (size_t)r * N + c));
                    *(u32x2 *)(Wb + (size_t)r * N + c) = u32x2{bf16_pack(x[0], x[1]), bf16_pack(x[2], x[3])};
                }
            }
    }
};

// Bound by a compute unit's vector memory path, which the slabs (32 KB each, from L2) and the master weights (160 KB a tile, read
// and written) pass one after the other: two workgroups per compute unit take 15.1 us and 1.04 us per slab for a tile each, while the
// traffic of the weights alone takes 13.5 at the copy rate.  4 jobs x 500 rows (588 MB): 164 us; master weights requested behind the multiplies 177; the
// register kernel, whose wavefronts read H and G from L2 once per 64 x 64 block, 204.  Four wavefronts that multiply and four that
// update, the sums handed over in LDS: 176 us (98 without the weights' traffic, 119 with the stores only, 110 with the loads
// only).  64 x 128 tiles, two or three per compute unit: step 11 - 17 us longer.
__global__ __launch_bounds__(256, 2) void grouped_dw_sgd_tiled(UpdateArgs a)
{
    using T = TileMfma<kDwTile, kDwTile, 2, 2, true, true>;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[T::kLds];
    dw_mean_loss(a, gridDim.x - 1 - blockIdx.x);      // the last workgroups have a tile less than the first
    const UpdateWalk walk(a);
    T::run(walk, smem);
}

static hipError_t launch_dw_tiled(const UpdateWithLoss *p, uint32_t n, hipStream_t stream, uint64_t *launches)
{
    for (uint32_t at = 0; at < n; at += kMaxProblems) {
        UpdateArgs a{};
        const uint64_t tiles = fill_updates(a, p + at, std::min(kMaxProblems, n - at), [](const UpdateProblem &q) {
            return (uint64_t)((q.K + kDwTile - 1) / kDwTile) * ((q.N + kDwTile - 1) / kDwTile);
        });
        if (tiles == 0) continue;
        if (tiles > 0x7fffffffull) return hipErrorInvalidValue;
        hipLaunchKernelGGL(grouped_dw_sgd_tiled, dim3((uint32_t)std::min<uint64_t>(tiles, 2 * resident_grid())), dim3(256), 0, stream, a);
        if (launches) *launches += 1;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_grouped_dw_sgd(const UpdateWithLoss *p, uint32_t n, bool cached, hipStream_t stream,
                                 uint64_t *launches)
{
    // One kernel for all updates of a step (two would each ramp up and drain): the tiled one if a weight's rows, on
    // average over the weights, are at least 192.  Register / tiled, step of 8 jobs of 2048-wide layers at 130 / 160 / 192 / 224 rows: 408 /
    // 428 / 445 / 466 us, 412 / 420 / 431 / 442 us; 4 jobs of 1024 - 1536 - 776 at 130 / 160 / 200 rows: 79 / 80 / 85, 81 / 82 / 83.
    double rows = 0, weights = 0;
    bool fits = true;
    for (uint32_t i = 0; i < n; ++i) {
        const double w = (double)p[i].K * p[i].N;
        weights += w;
        rows += w * p[i].M;
        fits = fits && p[i].K < kTiledMaxWidth && p[i].N < kTiledMaxWidth;
    }
    if (fits && rows >= kDwTiledRows * weights) return launch_dw_tiled(p, n, stream, launches);
    // 32 x 64 blocks of few rows against 64 x 64, steps of 16 sets of jobs (4 - 8 jobs of two to five layers of 128 - 2048): weights from HBM at 64 / 88 / 104 / 128
    // rows 0.970 / 0.968 / 0.960 / 0.985 of the time on average, at 150 and 180 rows slower in four sets of five; from the cache at 48 / 64 / 88 rows 0.956 / 0.974 /
    // 0.972, at 128 slower in two of four.  The mean decides also where rows differ: 7 jobs x 8 rows and one x 500, 1824 - 1480 - 152, 118 / 130 us.
    // Slower within these limits and known: 8 jobs of 872 - 2032 - 872 - 528 - 128, whose second layer is two whole rounds of 64 x 64 blocks, at 64 and 88 rows from the
    // cache 124 / 122 and 134 / 131, at 128 rows from HBM 162 / 157; 4 jobs of 680 - 1888 - 1336 - 1952 - 784, by up to 1 %.
    // And not where 64 x 64 blocks are all under way at once: 2 jobs of 744 - 2040 - 600 - 840 - 136 at 48 / 72 / 96 rows 66 / 69 / 71, 65 / 68 / 68.
    uint64_t tall_tiles = 0;
    for (uint32_t i = 0; i < n; ++i) tall_tiles += (uint64_t)((p[i].K + kUpdK - 1) / kUpdK) * ((p[i].N + kUpdN - 1) / kUpdN);
    const bool few_rows = rows <= (cached ? 88 : 128) * weights && tall_tiles > 2 * resident_grid();
    const uint32_t tile_k = few_rows ? kUpdFewK : kUpdK;
    for (uint32_t at = 0; at < n; at += kMaxProblems) {
        UpdateArgs a{};
        const uint64_t tiles = fill_updates(a, p + at, std::min(kMaxProblems, n - at), [&](const UpdateProblem &q) {
            return (uint64_t)((q.K + tile_k - 1) / tile_k) * ((q.N + kUpdN - 1) / kUpdN);
        });
        if (tiles == 0) continue;
        if (tiles > 0x7fffffffull) return hipErrorInvalidValue;
        hipLaunchKernelGGL(few_rows ? grouped_dw_sgd_few_rows : grouped_dw_sgd, dim3((uint32_t)tiles), dim3(256), 0, stream, a);
        if (launches) *launches += 1;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace salus
