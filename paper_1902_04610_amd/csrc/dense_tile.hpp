// One output tile of a dense layer, computed by a workgroup of four wavefronts:
// the arithmetic shared by the per-depth grouped kernels and the depth-fused ones.
#pragma once
#include "group.hpp"

namespace salus {

// Combine the four wavefronts' partial tiles.  Accumulator register r (0..3)
// of every 16x16 block holds row 4*(lane/16)+r, so wavefront w ends up owning
// rows with r == w: each wavefront sends the other three quarters through LDS
// and adds what it receives in a fixed order.
template <int NACC>
__device__ inline void reduce_scatter(f32x4 (&acc)[NACC], float (&own)[NACC], float *lds)
{
    constexpr int G = NACC < 16 ? NACC : 16;    // accumulators per pass (bounds the LDS footprint)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // lds[dst wave][source slot][accumulator in pass][lane]
#pragma unroll
    for (int base = 0; base < NACC; base += G) {
        if (base) __syncthreads();              // the previous pass has been read
#pragma unroll
        for (int d = 0; d < kWaves; ++d) {
            if (d == wave) continue;
            const int slot = (wave - d - 1) & 3;
            float *to = lds + ((d * 3 + slot) * G) * 64 + lane;
#pragma unroll
            for (int i = 0; i < G; ++i) to[i * 64] = acc[base + i][d];
        }
        __syncthreads();
        const float *from = lds + (wave * 3 * G) * 64 + lane;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const f32x4 mine = acc[base + i];
            float v = wave == 0 ? mine[0] : wave == 1 ? mine[1] : wave == 2 ? mine[2] : mine[3];
            v += from[(0 * G + i) * 64];
            v += from[(1 * G + i) * 64];
            v += from[(2 * G + i) * 64];
            own[base + i] = v;
        }
    }
}

template <int NACC>
constexpr int reduce_lds_floats() { return kWaves * 3 * (NACC < 16 ? NACC : 16) * 64; }

// ---------------------------------------------------------------------------
// bf16 weights and activations, float accumulation, v_mfma_f32_16x16x32_bf16.
// Tile: TM = 16*MT rows x 128 columns.  Lane (c = lane%16, g = lane/16) of a
// wavefront loads, per k-step of 32 rows, the 8x8 block W[k0+8g .. +7][n0+8c ..
// +7] (eight 16-byte loads, 256 contiguous bytes per row across the 16 lanes)
// and transposes it in registers; column i of the block is the B operand of
// MFMA i, whose 16 output columns are n0 + 8c + i.  The A operand is
// X[m0 + c][k0+8g .. +7].  Both operands use the same 8 k-values per lane
// group, which is all the MFMA contraction needs.
// TW (backward pass, dX = dY . W^T): W is stored N x K, so the eight k-values of
// output column n0+8c+i are contiguous in row n0+8c+i and are loaded as they are.
// ---------------------------------------------------------------------------
// NT: every weight is read by one workgroup only (each job has a single row tile),
// so the loads carry the non-temporal hint and do not displace activations in
// L2.  With several row tiles per column tile the neighbours read the same
// weights at about the same time and a plain load lets the second one hit in L2.
// CPL: columns per lane, 8, 4 or 2; the tile is 16 * CPL columns wide.  An output's products are summed in the same order
// whatever the width, so the result is the same to the bit.  D: k-steps in flight per wavefront; a narrow tile has fewer
// bytes per step and needs more of them to cover the latency.
template <int MT, bool TW, bool NT, int CPL = 8, int D = 2>
__device__ inline void dense_bf16_tile(const Problem &p, const Tile tile, float *lds)
{
    constexpr int NACC = MT * CPL, NROW = TW ? CPL : 8;      // weight vectors per lane and k-step
    typedef unsigned int wvec __attribute__((ext_vector_type(TW ? 4 : CPL / 2)));
    const uint32_t M = p.M, K = p.K, N = p.N;
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t ncol = tile.n0 + CPL * c;
    const bool col_ok = ncol < N;
    const Global<uint16_t> *W = (const Global<uint16_t> *)p.W;
    const Global<uint16_t> *X = (const Global<uint16_t> *)p.X;

    f32x4 acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nsteps = (int)((K + 31) / 32);
    const u32x4 zero = {0u, 0u, 0u, 0u};

    // Loads are never predicated: a lane whose block lies outside the matrix
    // reads a clamped, valid address instead and its values are dropped later
    // (rows >= M and columns >= N are never stored; k-groups >= K get a zero A
    // operand).  With no branch around any load the compiler can count exactly
    // how many loads may stay in flight at each use, which is what keeps the
    // next step's loads outstanding while this step is multiplied.
    const uint32_t ncol_c = col_ok ? ncol : 0u;
    // Row-major W: row pitch N.  Strip layout: the 128 columns of this tile are one
    // contiguous K x 128 block (pitch 128), so a wavefront's k-step is 8 KB in one piece.
    const bool blocked_in = !TW && (p.flags & kInBlocked);     // implies M <= 32, so tile.m0 == 0
    const uint32_t xtiles = (M + 15) / 16;
    const bool strip = !TW && (p.flags & kStripW);
    const uint32_t wpitch = strip ? 128u : N;
    const Global<uint16_t> *Wc = strip ? W + (size_t)(tile.n0 & ~127u) * K + (tile.n0 & 127u) + CPL * c : W + ncol_c;
    auto load = [&](int s, wvec (&w)[NROW], u32x4 (&x)[MT], bool &k_ok) {
        const uint32_t kb = 32u * (uint32_t)s + 8u * (uint32_t)g;
        k_ok = kb < K;
        const uint32_t kc = k_ok ? kb : 0u;
#pragma unroll
        for (int r = 0; r < NROW; ++r) {
            const Global<uint16_t> *at = TW ? W + (size_t)(ncol_c + r) * K + kc : Wc + (size_t)(kc + r) * wpitch;
            w[r] = NT ? __builtin_nontemporal_load((const Global<wvec> *)at) : *(const Global<wvec> *)at;
        }
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            if (blocked_in) {
                // one contiguous kilobyte per wavefront; a row tile the job does not
                // have (its rows are never stored) reads the job's last one instead
                const uint32_t tt = (uint32_t)t < xtiles ? (uint32_t)t : xtiles - 1;
                x[t] = *(const Global<u32x4> *)(X + (((size_t)(kc >> 5) * xtiles + tt) * 64 + lane) * 8);
            } else {
                const uint32_t row = tile.m0 + 16 * t + c;
                x[t] = *(const Global<u32x4> *)(X + (size_t)(row < M ? row : M - 1) * K + kc);
            }
        }
    };
    auto compute = [&](const wvec (&w)[NROW], const u32x4 (&xr)[MT], bool k_ok) {
        u32x4 x[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) x[t] = k_ok ? xr[t] : zero;
        // Narrow tiles drop the weights of k-groups >= K as well (a selector of 0x0c is a zero byte): an infinite one, which a lane reads again there, times
        // zero would be a NaN.  LDS tiles, whose jobs these take when they are few, fetch zeros for both.
        const bool drop = !TW && CPL < 8 && !k_ok;
        const uint32_t even = drop ? 0x0c0c0c0cu : 0x05040100u, odd = drop ? 0x0c0c0c0cu : 0x07060302u;
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
            // column i of the 8 x CPL block: dword j = (row 2j, row 2j+1)
            u32x4 b;
            if constexpr (TW) {
                b = NT || k_ok ? w[i] : zero;      // several row tiles: dropped too (the ring, which has such jobs when they are more, fetches zeros)
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    b[j] = __builtin_amdgcn_perm(w[2 * j + 1][i >> 1], w[2 * j][i >> 1], (i & 1) ? odd : even);
            }
#pragma unroll
            for (int t = 0; t < MT; ++t)
                acc[t * CPL + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8, x[t]), __builtin_bit_cast(bf16x8, b), acc[t * CPL + i],
                    0, 0, 0);
        }
    };

    // The four wavefronts take k-steps wave, wave+4, ...: this wavefront owns
    // `mine` steps.  D steps are in flight at any time; the last (fewer than 2 D)
    // steps are peeled so that the main loop never loads past the end.
    const int mine = nsteps > wave ? (nsteps - wave + kWaves - 1) / kWaves : 0;
    auto step = [&](int i) { return wave + kWaves * i; };
    if constexpr (D == 2) {
        // Not the loop below with D = 2: in that form the 64-row tile (MT = 4, capped at 256 registers) spills 11 of them, and a reload
        // inside the loop waits for all weights in flight (64 models x 48 / 64 rows of 1024 - 4096 - 1024 - 1024: 292 / 308 us
        // a round against 251 / 270 us in this form, which just fits).
        wvec w0[NROW], w1[NROW];
        u32x4 x0[MT], x1[MT];
        bool ok0, ok1;
        load(step(0), w0, x0, ok0);
        load(step(1), w1, x1, ok1);
        int i = 0;
        for (; i + 3 < mine; i += 2) {
            // keep the instruction scheduler from sinking the loads below the next
            // multiply phase: each phase must stay where it is written
            compute(w0, x0, ok0);
            __builtin_amdgcn_sched_barrier(0);
            load(step(i + 2), w0, x0, ok0);
            __builtin_amdgcn_sched_barrier(0);
            compute(w1, x1, ok1);
            __builtin_amdgcn_sched_barrier(0);
            load(step(i + 3), w1, x1, ok1);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int left = mine - i;
        if (left >= 1) compute(w0, x0, ok0);
        if (left == 3) load(step(i + 2), w0, x0, ok0);
        if (left >= 2) compute(w1, x1, ok1);
        if (left == 3) compute(w0, x0, ok0);
    } else {
        wvec w[D][NROW];
        u32x4 x[D][MT];
        bool ok[D];
#pragma unroll
        for (int d = 0; d < D; ++d) load(step(d), w[d], x[d], ok[d]);
        int i = 0;
        for (; i + 2 * D <= mine; i += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                compute(w[d], x[d], !NT || ok[d]);      // the last step of a wavefront, the only one that can end past K, is peeled
                __builtin_amdgcn_sched_barrier(0);
                load(step(i + d + D), w[d], x[d], ok[d]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const int left = mine - i;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (d < left) compute(w[d], x[d], ok[d]);
            if (d + D < left) load(step(i + d + D), w[d], x[d], ok[d]);
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d + D < left) compute(w[d], x[d], ok[d]);
    }

    float own[NACC];
    reduce_scatter<NACC>(acc, own, lds);

    const uint32_t act = p.flags & 0xffu;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const uint32_t row = tile.m0 + 16 * t + 4 * g + wave;
        if (row >= M || !col_ok) continue;
        float v[CPL];
#pragma unroll
        for (int i = 0; i < CPL; ++i) v[i] = activate(own[t * CPL + i], act);
        typedef unsigned int out_vec __attribute__((ext_vector_type(CPL / 2)));
        if (p.flags & kMaskPositive) {
            // ReLU derivative taken from the stored bf16 activation (sign bit clear, not zero)
            const out_vec h = *(const Global<out_vec> *)((const Global<uint16_t> *)p.aux + (size_t)row * N + ncol);
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                const uint32_t bits = (h[i >> 1] >> ((i & 1) * 16)) & 0xffffu;
                if ((bits & 0x8000u) || !(bits & 0x7fffu)) v[i] = 0.0f;
            }
        }
        if (p.flags & kOutBf16) {
            out_vec o;
#pragma unroll
            for (int j = 0; j < CPL / 2; ++j) o[j] = bf16_pack(v[2 * j], v[2 * j + 1]);
            if (p.flags & kOutBlocked) {
                // these columns are in k-group (ncol / 8) % 4 of k-step ncol / 32 of the next layer
                const size_t unit = (((size_t)(ncol >> 5) * xtiles + (row >> 4)) * 4 + ((ncol >> 3) & 3)) * 16 +
                                    (row & 15);
                *(Global<out_vec> *)((Global<uint16_t> *)p.Y + unit * 8 + (ncol & 7u)) = o;
            } else {
                *(Global<out_vec> *)((Global<uint16_t> *)p.Y + (size_t)row * N + ncol) = o;
            }
        } else {
            Global<float> *y = (Global<float> *)p.Y + (size_t)row * N + ncol;
            if constexpr (CPL == 2) {
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                *(Global<f32x2> *)y = f32x2{v[0], v[1]};
            } else {
#pragma unroll
                for (int j = 0; j < CPL; j += 4) *(Global<f32x4> *)(y + j) = f32x4{v[j], v[j + 1], v[j + 2], v[j + 3]};
            }
        }
    }
}

// ---------------------------------------------------------------------------
// float weights and activations, v_mfma_f32_16x16x4_f32 (true fp32 products).
// Tile: 16*MT rows x 64 columns; a k-step covers 16 rows of W.  Lane (c, g)
// loads W[k0+4g+q][n0+4c .. +3] for q = 0..3 and X[m0+c][k0+4g .. +3]; MFMA
// (q, i) multiplies component q of X with component i of W row q, so lane
// group g contributes k = k0+4g+q in step q and output column n0+4c+i.
// ---------------------------------------------------------------------------
// D: k-steps in flight per wavefront, CPL: columns per lane (4 or 1; the tile is 16 * CPL wide), as above.
template <int MT, int D = 2, int CPL = 4>
__device__ inline void dense_f32_tile(const Problem &p, const Tile tile, float *lds)
{
    constexpr int NACC = MT * CPL;
    typedef float wvec __attribute__((ext_vector_type(CPL)));
    const uint32_t M = p.M, K = p.K, N = p.N;
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t ncol = tile.n0 + CPL * c;
    const bool col_ok = ncol < N;
    const Global<float> *W = (const Global<float> *)p.W;
    const Global<float> *X = (const Global<float> *)p.X;

    f32x4 acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nsteps = (int)((K + 15) / 16);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

    // unpredicated loads from clamped addresses, as in the bf16 kernel
    const uint32_t ncol_c = col_ok ? ncol : 0u;
    auto load = [&](int s, wvec (&w)[4], f32x4 (&x)[MT], bool &k_ok) {
        const uint32_t kb = 16u * (uint32_t)s + 4u * (uint32_t)g;
        k_ok = kb < K;
        const uint32_t kc = k_ok ? kb : 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = *(const Global<wvec> *)(W + (size_t)(kc + q) * N + ncol_c);
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const uint32_t row = tile.m0 + 16 * t + c;
            x[t] = *(const Global<f32x4> *)(X + (size_t)(row < M ? row : M - 1) * K + kc);
        }
    };
    auto compute = [&](const wvec (&w)[4], const f32x4 (&xr)[MT], bool k_ok) {
        f32x4 x[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) x[t] = k_ok ? xr[t] : zero;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < CPL; ++i)
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    acc[t * CPL + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t][q], w[q][i], acc[t * CPL + i], 0, 0, 0);
    };

    const int mine = nsteps > wave ? (nsteps - wave + kWaves - 1) / kWaves : 0;
    auto step = [&](int i) { return wave + kWaves * i; };
    if constexpr (D == 2) {
        wvec w0[4], w1[4];
        f32x4 x0[MT], x1[MT];
        bool ok0, ok1;
        load(step(0), w0, x0, ok0);
        load(step(1), w1, x1, ok1);
        int i = 0;
        for (; i + 3 < mine; i += 2) {
            // keep the instruction scheduler from sinking the loads below the next
            // multiply phase: each phase must stay where it is written
            compute(w0, x0, ok0);
            __builtin_amdgcn_sched_barrier(0);
            load(step(i + 2), w0, x0, ok0);
            __builtin_amdgcn_sched_barrier(0);
            compute(w1, x1, ok1);
            __builtin_amdgcn_sched_barrier(0);
            load(step(i + 3), w1, x1, ok1);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int left = mine - i;
        if (left >= 1) compute(w0, x0, ok0);
        if (left == 3) load(step(i + 2), w0, x0, ok0);
        if (left >= 2) compute(w1, x1, ok1);
        if (left == 3) compute(w0, x0, ok0);
    } else {
        wvec w[D][4];
        f32x4 x[D][MT];
        bool ok[D];
#pragma unroll
        for (int d = 0; d < D; ++d) load(step(d), w[d], x[d], ok[d]);
        int i = 0;
        for (; i + 2 * D <= mine; i += D) {
            // keep the instruction scheduler from sinking the loads below the next
            // multiply phase: each phase must stay where it is written
#pragma unroll
            for (int d = 0; d < D; ++d) {
                compute(w[d], x[d], ok[d]);
                __builtin_amdgcn_sched_barrier(0);
                load(step(i + d + D), w[d], x[d], ok[d]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const int left = mine - i;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (d < left) compute(w[d], x[d], ok[d]);
            if (d + D < left) load(step(i + d + D), w[d], x[d], ok[d]);
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d + D < left) compute(w[d], x[d], ok[d]);
    }

    float own[NACC];
    reduce_scatter<NACC>(acc, own, lds);

    const uint32_t act = p.flags & 0xffu;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const uint32_t row = tile.m0 + 16 * t + 4 * g + wave;
        if (row >= M || !col_ok) continue;
        wvec o;
#pragma unroll
        for (int i = 0; i < CPL; ++i) o[i] = activate_f32(own[t * CPL + i], act);
        *(Global<wvec> *)((Global<float> *)p.Y + (size_t)row * N + ncol) = o;
    }
}

}  // namespace salus
