// Tiles of a dense layer for launches with fewer tiles of 128 columns than compute units (16, 32 or 64 columns), or with so few that
// their number does not divide evenly (64 - 128): the arithmetic of dense_bf16_tile, in the same order, with its operands fetched straight
// into LDS.
#pragma once
#include <type_traits>
#include <utility>

#include "dense_tile.hpp"
#include "tile_mfma.hpp"

namespace salus {

// What a launch of few workgroups lasts is how long one compute unit fetches one tile, and what bounds that is not bytes but
// vector memory instructions: a lane that is to hold a column of a narrow tile loads 4 bytes of each row and no more, a quarter
// of what the instruction can fetch.  So weights travel in
// the order in which they lie in memory, a kilobyte an instruction, into an LDS ring that each wavefront has to itself (no
// barrier in the loop), and ds_read_b64_tr_b16 hands each lane its column.  One job, one row,
// 1024 -> 4096 -> 1024 -> 1024: 15.7 us, 24.0 with loads into registers; 2048 -> 1024 4.0 / 9.2; 3 jobs x 32 rows, 4096 -> 1024 14.8 / 22.
// 16 * NB columns, 16 * MT rows; D k-steps of 32 in flight per wavefront, as many as BUDGET bytes of LDS hold, STEP of which share a
// wait.  STEP == 1 is for half the LDS, two workgroups per compute unit: the sums take the ring's place there.
template <int MT, int NB, int STEP = 2, uint32_t BUDGET = 160 * 1024>
struct NarrowTile {
    static constexpr uint32_t kRequests = NB + MT, kSlot = kRequests * 1024;       // instructions and bytes of a k-step
    static constexpr int kNacc = MT * NB;
    static constexpr uint32_t kSums = reduce_lds_floats<kNacc>() * 4;
    static constexpr bool kAlias = STEP == 1;
    static constexpr uint32_t kWant = NB + MT <= 2 ? 16 : 8, kRoom = BUDGET - (kAlias ? 0 : kSums);
    static constexpr uint32_t D = kWant * kSlot * kWaves <= kRoom ? kWant : kRoom / (kSlot * kWaves) / STEP * STEP;
    static constexpr uint32_t kRing = D * kSlot, kSumsAt = kAlias ? 0 : kWaves * kRing, kLds = kAlias ? (kSums > kWaves * kRing ? kSums : kWaves * kRing) : kWaves * kRing + kSums;
    static_assert(D >= 2 * STEP && (D - STEP) * kRequests <= 63, "largest count of s_waitcnt");

    // Where the transposing reads find a k-row: its row in the slot (an involution), and what is xored to the number of its
    // 16-byte chunks.  Such a read touches rows 8 g .. 8 g + 3 of all four g, 32 bytes each, which are spread evenly over
    // the 256 bytes that LDS delivers at a time.
    __device__ static uint32_t row_at(uint32_t r) { return NB == 1 ? r ^ ((r >> 3 & 1u) << 2) : r; }
    __device__ static uint32_t chunk_swizzle(uint32_t r)
    {
        return NB == 2 ? (r >> 3 & 1u) << 1 : NB == 4 ? (r >> 1 & 1u) << 1 | (r >> 3 & 1u) << 2 : NB == 8 ? (r & 3u) << 1 | (r >> 3 & 1u) << 3 : 0u;
    }

    // The last D / STEP groups of k-steps, of which `groups` are there.
    template <size_t... I, typename Multiply>
    __device__ static void drain(std::index_sequence<I...>, uint32_t groups, Multiply &multiply)
    {
        auto one = [&](auto behind) {
            constexpr uint32_t kBehind = decltype(behind)::value;
            if (groups <= kBehind) return;
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBehind * STEP * kRequests) : "memory");
            multiply(false);
        };
        (one(std::integral_constant<uint32_t, sizeof...(I) - 1 - I>{}), ...);
    }

    __device__ static void run(const Problem &p, const Tile tile, unsigned char *smem)
    {
        const uint32_t M = p.M, K = p.K, N = p.N;
        const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const bool blocked_in = (p.flags & kInBlocked) != 0, strip = (p.flags & kStripW) != 0;
        const uint32_t xtiles = (M + 15) / 16;

        // Requests of a k-step: NB kilobytes of weights, 32 / NB rows each, then a kilobyte of activations per row tile.
        constexpr uint32_t kLanes = 2 * NB;      // lanes of a k-row
        const uint32_t pitch = strip ? 256u : N * 2u;
        const uint32_t first_col = strip ? (tile.n0 & 127u) : tile.n0;
        uint32_t w_off[NB], krow[NB];
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)NB; ++i) {
            const uint32_t at = 64u * i + lane;
            krow[i] = row_at(at / kLanes);
            const uint32_t col = 8u * ((at % kLanes) ^ chunk_swizzle(krow[i]));
            w_off[i] = tile.n0 + col < N ? krow[i] * pitch + (first_col + col) * 2u + (strip && first_col + col >= 128u ? (K - 1) * 256u : 0u) : kOutside;
        }
        uint64_t w_base = (uint64_t)(uintptr_t)p.W + (strip ? (uint64_t)(tile.n0 & ~127u) * K * 2u : 0);
        uint64_t x_base = (uint64_t)(uintptr_t)p.X;
        uint32_t x_off[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            // a row tile that the job does not have (its rows are never stored) reads the last one instead
            const uint32_t row = tile.m0 + 16u * t + c, tt = min((uint32_t)t, xtiles - 1);
            x_off[t] = blocked_in ? tt * 1024u + 16u * lane : (row < M ? row : M - 1) * K * 2u + 16u * g;
        }
        const uint64_t w_step = (uint64_t)32u * pitch, x_step = blocked_in ? xtiles * 1024u : 64u;
        const uint32_t nsteps = (K + 31) / 32;
        w_base = uniform64(w_base + (uint64_t)wave * w_step);
        x_base = uniform64(x_base + (uint64_t)wave * x_step);
        uint32_t k = 32u * wave;                 // first k-row of the next request
        const uint32_t ring = lds_address(smem) + wave * kRing;
        uint32_t to = 0;
        // rows from K on arrive as zeros, without a memory access; so does every step past the last
        auto request = [&]() {
            const int left = (int)K - (int)k;
#pragma unroll
            for (uint32_t i = 0; i < (uint32_t)NB; ++i)
                dma16(ring + to + i * 1024u, w_base, (int)krow[i] < left ? w_off[i] : kOutside);
#pragma unroll
            for (int t = 0; t < MT; ++t) dma16(ring + to + (NB + t) * 1024u, x_base, 8 * g < left ? x_off[t] : kOutside);
            k += 32u * kWaves;
            w_base += kWaves * w_step;
            x_base += kWaves * x_step;
            to = to + kSlot == kRing ? 0u : to + kSlot;
        };
        const uint32_t mine = nsteps > (uint32_t)wave ? (nsteps - wave + kWaves - 1) / kWaves : 0;
        uint32_t groups = (mine + STEP - 1) / STEP;        // of k-steps that share a wait; one past the last is all zeros
#pragma unroll 1
        for (uint32_t d = 0; d < min(groups, D / STEP); ++d)
#pragma unroll
            for (int s = 0; s < STEP; ++s) request();

        f32x4 acc[kNacc];
#pragma unroll
        for (int i = 0; i < kNacc; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        const unsigned char *from = smem + wave * kRing;
        // transposing reads: the 16 lanes of group g take four k-rows x 16 columns from row 8 g (and four more), four lanes a row
        uint32_t at_w[2][NB];
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h)
#pragma unroll
            for (uint32_t j = 0; j < (uint32_t)NB; ++j) {
                const uint32_t r = 8u * g + 4u * h + (c >> 2);
                at_w[h][j] = row_at(r) * (32u * NB) + ((2u * j) ^ chunk_swizzle(r)) * 16u + 8u * (c & 3);
            }
        uint32_t at = 0;
        auto multiply = [&](bool more) {
            bf16x8 x[STEP][MT], w[STEP][NB];
#pragma unroll
            for (int s = 0; s < STEP; ++s) {
                const unsigned char *slot = from + at + s * kSlot;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    typedef __attribute__((address_space(3))) s16x4 *lds_t;
                    struct { s16x4 lo, hi; } v;
                    v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(slot + at_w[0][j]));
                    v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(slot + at_w[1][j]));
                    w[s][j] = __builtin_bit_cast(bf16x8, v);
                }
#pragma unroll
                for (int t = 0; t < MT; ++t) x[s][t] = *(const bf16x8 *)(slot + (NB + t) * 1024 + 16 * lane);
            }
            if (more) {
                // the slots have been read before they are requested into
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int s = 0; s < STEP; ++s) request();
            }
#pragma unroll
            for (int s = 0; s < STEP; ++s)
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int t = 0; t < MT; ++t) acc[t * NB + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[s][t], w[s][j], acc[t * NB + j], 0, 0, 0);
            at = at + STEP * kSlot == kRing ? 0u : at + STEP * kSlot;
        };
#pragma unroll 1
        for (; groups > D / STEP; --groups) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - STEP) * kRequests) : "memory");
            multiply(true);
        }
        // the last ones, all requested: nothing is left in flight after them
        drain(std::make_index_sequence<D / STEP>{}, groups, multiply);

        float own[kNacc];
        if (kAlias) __syncthreads();
        reduce_scatter<kNacc>(acc, own, (float *)(smem + kSumsAt));
        const uint32_t act = p.flags & 0xffu;
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const uint32_t row = tile.m0 + 16 * t + 4 * g + wave, n = tile.n0 + 16 * j + c;
                if (row >= M || n >= N) continue;
                const float v = activate(own[t * NB + j], act);
                if (!(p.flags & kOutBf16)) {
                    ((Global<float> *)p.Y)[(size_t)row * N + n] = v;
                } else {
                    // blocked: column n is in k-group (n / 8) % 4 of k-step n / 32 of the next layer
                    const size_t unit = (((size_t)(n >> 5) * xtiles + (row >> 4)) * 4 + ((n >> 3) & 3)) * 16 + (row & 15);
                    ((Global<uint16_t> *)p.Y)[p.flags & kOutBlocked ? unit * 8 + (n & 7u) : (size_t)row * N + n] = (uint16_t)bf16_bits(v);
                }
            }
    }
};

}  // namespace salus
