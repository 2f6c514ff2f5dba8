// Compute-bound tiles: C[m][n] = sum over k of M-side(m, k) * N-side(n, k) for one BM x BN tile, bf16
// operands, float sums, v_mfma_f32_32x32x16_bf16, operands streamed HBM -> LDS -> registers.
//
// What bounds it: the matrix pipes, if everything else stays out of their way.  So
//   - operands go from memory straight into LDS (buffer_load_dwordx4 .. lds): no staging registers, no LDS
//     stores, no address arithmetic in the loop (a scalar base that advances per slab + fixed 32-bit offsets, which the launcher keeps below 2 GB);
//   - an operand whose contraction index is not its contiguous one (the K x N weights of a forward pass;
//     both operands of H^T . G) is stored in LDS as it lies in memory and transposed on the way to the
//     registers by ds_read_b64_tr_b16, instead of in registers on the way in;
//   - the contraction is walked in slabs of 64, four k-steps of 16.  The fragments of a k-step are read while the step
//     before it is multiplied, one read after each multiply; requests are spread over the k-steps the same way.
//   - what a wait costs is how late its request was issued, so LDS holds as much of the future as fits: a "major"
//     operand (below) three slabs, a "tr" operand two slabs that are freed and refilled in halves of 32 k-rows.
//     Either way a request has four k-steps (2048 cycles of the matrix pipe) after the last of its kind is issued.
//     One barrier before every odd k-step says at once: what the next reads need has landed (vmcnt leaves
//     the last slab's worth of requests in flight), and what will be overwritten has been read.
//   - the request stream does not stop at the end of a tile: a workgroup walks its tiles (one or two
//     workgroups per compute unit) and the next tile's first slabs travel during the epilogue.
// The M side is the second MFMA operand, so a lane owns one row m (lane % 32) and runs of four consecutive columns
// n.  Stored like that, an instruction would touch 32 lines with 32 bytes each and the L2's request rate
// would bound the epilogue; to_lines_* trade register bits for lane bits so that a store writes 8 whole lines.
//
// LDS layout.  An operand with contiguous contraction index ("major"): line r = its row r, 64 k-values =
// eight 16-byte chunks, chunk c at c ^ (r / 2 & 7): sixteen consecutive rows of a fragment read (256 bytes, what LDS
// delivers per cycle) fall into different banks.  Transposed ("tr"): line r = k-row r of the slab, chunk c (8
// columns) at c ^ 4 * (r & 3), of 64-column tiles c ^ 4 * (r / 2 & 1): the four k-rows x 64 bytes that 32 lanes of a transposing read touch fall into the
// four quarters of the 256-byte bank row.
// The DMA writes LDS linearly, so the permutation is applied to the source address, inside a 128-byte line.
//
// Ragged shapes.  Rows and columns outside the matrices and chunks beyond the end of the contraction (on both sides) are
// requested outside the buffer's range: they arrive as zeros without a memory access, and infinities and NaNs
// elsewhere in the operands cannot leak into the sums.
#pragma once
#include "group.hpp"

namespace salus {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kSlab = 64;            // contraction depth of a slab
constexpr uint32_t kMinSlabs = 3;         // a tile is walked in at least so many (the request stream runs two slabs
                                          // ahead and must not cross two tile ends at once); the extra ones are zeros

__device__ inline uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}

// The same lane number, computed here: keeps what is derived from it from being hoisted out of the slab loop, where
// every register is spoken for.
__device__ inline int fresh_lane()
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

// 16 bytes per lane from base + off to LDS at `to` + 16 * lane; zeros where off is kOutside.  A raw buffer descriptor of
// 2 GB: the hardware's range check is the mask of the contraction's tail.
constexpr uint32_t kOutside = 0x80000000u;
// m0 (the LDS address) is reserved: the compiler sets it where it needs it and keeps nothing there, but it may take two
// equal settings for one unless it knows that the register changes in between.  It warns about any reserved register.
// ONCE: non-temporal, for what no other workgroup will ask for.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool ONCE = false>
__device__ inline void dma16(uint32_t to, uint64_t base, uint32_t off)
{
    const u32x4 buffer = {(uint32_t)base, (uint32_t)(base >> 32) & 0xffffu, kOutside, 0x00027000u};
    if constexpr (ONCE) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"s"(to), "v"(off), "s"(buffer) : "m0", "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(to), "v"(off), "s"(buffer) : "m0", "memory");
}
#pragma clang diagnostic pop

__device__ inline uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (uint64_t)hi << 32 | lo;
}

// One operand as the tile walk sees it.
struct Operand {
    const void *ptr;
    uint64_t depth;       // contraction length
    uint32_t extent;      // rows (major) or columns (tr) of the matrix
    uint32_t pitch;       // bytes between rows (major) or between k-rows (tr)
    bool strip;           // tr only: columns in strips of 128, each depth x 128 contiguous
};

// tr: what is xored to the chunks of k-row `row` (64 columns: two k-rows share a 256-byte bank row)
template <int B>
__device__ inline uint32_t tr_swizzle(uint32_t row) { return B >= 128 ? 4u * (row & 3u) : 4u * ((row >> 1) & 1u); }

// One operand's request stream: where it is in the walk and what this wavefront's share of it is, I instructions of
// 1 KB per slab.  Requests are issued in k-steps 3, 0, 1, 2 (major: a slab, three slabs ahead) or 1, 2 and 3, 0 (tr: the
// first and the second half of a slab, two slabs ahead) of the slab being multiplied.
// UNIT: k-values of a stage (a major operand's is a whole slab, the 128 bytes of a line).  ONCE: requests are non-temporal.
template <int B, bool TR, int WAVES, int STAGES = TR ? 2 : 3, uint32_t UNIT = kSlab, bool ONCE = false>
struct OperandStream {
    static constexpr int kBytes = B * (int)UNIT * 2, I = kBytes / 1024 / WAVES;
    static constexpr int kStages = STAGES, kRing = kStages * kBytes;
    static constexpr int kHalf = I > 1 ? I / 2 : 1;
    static constexpr int kChunks = B / 8, kRowsPer = TR ? 64 / kChunks : 8;      // tr: 16-byte chunks of a k-row
    static_assert(I >= 1 && kBytes == I * 1024 * WAVES && (!TR || STAGES != 2 || I % 2 == 0), "whole instructions per wavefront");
    static_assert(UNIT == kSlab || (TR && STAGES != 2), "parts of a slab");
    uint64_t base;        // scalar: of the slab (unit) under the cursor
    uint64_t stride;      // bytes per slab (unit)
    uint32_t off[I];      // per lane
    uint32_t k, depth, slabs_left, at;      // at: offset in the ring of the stage it goes to; slabs_left: in units
    int lane_k;           // this lane's k-row (tr) or first k-value (major) in a request of piece 0

    __device__ void start(int lane)
    {
        at = 0;
        lane_k = TR ? lane / kChunks : (int)(8u * chunk_of((uint32_t)lane / 8u, lane));
    }
    // The KB of the slab that instruction i fetches: where a tr ring has two stages, instructions 0 .. I/2 - 1 cover the
    // k-rows below 32, the others the rest.
    __device__ static uint32_t piece(int wave, int i) { return TR && STAGES == 2 ? (uint32_t)((i / kHalf) * (WAVES * kHalf) + wave * kHalf + i % kHalf) : (uint32_t)(wave * I + i); }
    __device__ static uint32_t row_of(int wave, int i, int lane)
    {
        return kRowsPer * piece(wave, i) + (uint32_t)(TR ? lane / kChunks : lane / 8);
    }
    __device__ static uint32_t chunk_of(uint32_t row, int lane)
    {
        return TR ? ((uint32_t)(lane % kChunks) ^ tr_swizzle<B>(row)) : ((uint32_t)(lane & 7) ^ ((row >> 1) & 7u));
    }
    __device__ void locate(const Operand &o, uint32_t first, int wave)
    {
        const int lane = fresh_lane();
        uint64_t from;
        if (TR) {
            from = o.strip ? (uint64_t)(first >> 7) * o.depth * 256u + (first & 127u) * 2u : (uint64_t)first * 2u;
            stride = (uint64_t)UNIT * o.pitch;
        } else {
            from = (uint64_t)first * o.pitch;
            stride = kSlab * 2;
        }
        base = uniform64((uint64_t)(uintptr_t)o.ptr + from);
        stride = uniform64(stride);
        k = 0;
        depth = __builtin_amdgcn_readfirstlane((uint32_t)o.depth);
        slabs_left = __builtin_amdgcn_readfirstlane(max((depth + kSlab - 1) / kSlab, kMinSlabs) * (kSlab / UNIT));
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const uint32_t r = row_of(wave, i, lane), c = chunk_of(r, lane);
            if (TR) {
                off[i] = r * o.pitch + (o.strip ? (c >> 4) * (uint32_t)(o.depth * 256u) + (c & 15u) * 16u : c * 16u);
                if (first + 8u * c >= o.extent) off[i] = kOutside;
            } else {
                off[i] = first + r < o.extent ? r * o.pitch + c * 16u : kOutside;
            }
        }
    }
    // Instruction i of the slab under the cursor.  Chunks beyond the contraction (all of them once the walk is over: depth
    // is then 0) are zeros: no branch, and always the same number of requests in flight.
    __device__ void fetch(int i, uint32_t lds, int wave) const
    {
        const uint32_t pc = piece(wave, i);
        const int left = (int)(depth - k) - (TR ? (int)(kRowsPer * pc) : 0);          // k-rows or k-values from here on
        const int mine = TR ? lane_k : (int)((uint32_t)lane_k ^ (32u * (pc & 1u)));
        dma16<ONCE>(lds + at + pc * 1024u, base, mine < left ? off[i] : kOutside);
    }
    // the requests that belong to k-step q
    __device__ void request(int q, uint32_t lds, int wave) const
    {
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const int when = TR ? 1 + (i * 4) / I : 3 + (i * 4) / I;       // tr: 1, 2, 3, 4; major: 3, 4, 5, 6
            if ((when & 3) == q) fetch(i, lds, wave);
        }
    }
    __device__ void advance()
    {
        base += stride;
        k += UNIT;
        --slabs_left;
        at = at + kBytes == (uint32_t)kRing ? 0u : at + kBytes;
    }
    __device__ void stop()       // the walk is over
    {
        k = depth = 0;
        slabs_left = ~0u;
        stride = 0;
    }
};

// Fragments of F consecutive 32-wide blocks for k-step ks: lane l holds 8 k-values (from 16 * ks + 8 * (l / 32)) of
// row or column l % 32 of a block.
template <int B, bool TR, int F>
struct Fragments {
    static_assert(F == 1 || F == 2 || F == 4, "the swizzle flips the low two bits of a block's number");
    uint32_t at[TR ? F : 4];
    // first: first row / column of the wavefront's part of the tile (a multiple of 32 * F)
    __device__ void init(uint32_t first, int lane)
    {
        if (TR) {
            const uint32_t i = lane & 15u, rr = i >> 2, row = 8u * (lane >> 5) + rr;
            const uint32_t c = (first >> 3) + 2u * ((lane >> 4) & 1u) + ((i & 3u) >> 1);
#pragma unroll
            for (uint32_t j = 0; j < (uint32_t)F; ++j) at[j] = row * (B * 2u) + (((c + 4u * j) ^ tr_swizzle<B>(rr)) << 4) + 8u * (i & 1u);
        } else {
            const uint32_t r = first + (lane & 31u);
#pragma unroll
            for (uint32_t ks = 0; ks < 4; ++ks) at[ks] = r * 128u + (((2u * ks + (lane >> 5)) ^ ((r >> 1) & 7u)) << 4);
        }
    }
    __device__ bf16x8 read(const unsigned char *base, int ks, int block) const
    {
        if (TR) {
            const unsigned char *p = base + at[block] + ks * 16 * (B * 2);
            typedef __attribute__((address_space(3))) s16x4 *lds_t;
            struct { s16x4 lo, hi; } v;
            v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(p));
            v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(p + 4 * (B * 2)));
            return __builtin_bit_cast(bf16x8, v);
        }
        return *(const bf16x8 *)(base + at[ks] + block * 32 * 128);
    }
};

// BM x BN tile by WM x WN wavefronts; TRM / TRN: the M / N side is stored with its rows along the
// contraction.  Walk: tile id -> place, operands and epilogue:
//   uint32_t tiles(); Place place(id); Operand m(Place), n(Place);
//   begin(Place, Held, m, n, lane): before the first multiply; (m, n) is the wavefront's corner in the tile;
//   finish(Place, acc, Held, m, n, lane, landed): calls landed() before its first store.
// Place has m0, n0 and depth.  The grid has at most tiles() workgroups.
template <int BM, int BN, int WM, int WN, bool TRM, bool TRN>
struct TileMfma {
    static constexpr int kWavesT = WM * WN, kThreads = 64 * kWavesT;
    static constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
    using SM = OperandStream<BM, TRM, kWavesT>;
    using SN = OperandStream<BN, TRN, kWavesT>;
    static constexpr uint32_t kLds = SM::kRing + SN::kRing;
    static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
    static_assert(FM * FN > 1, "a k-step places its reads between its multiplies");
    static_assert(!TRM || TRN, "the M side meets the end of a tile no later than the N side");
    typedef f32x16 Acc[FN][FM];

    template <typename Walk>
    __device__ static void run(const Walk &walk, unsigned char *smem)
    {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t wm = wave / WN, wn = wave % WN;
        const uint32_t lds_m = lds_address(smem), lds_n = lds_m + SM::kRing;
        Fragments<BM, TRM, FM> fm;
        Fragments<BN, TRN, FN> fn;
        fm.init(wm * (32u * FM), lane);
        fn.init(wn * (32u * FN), lane);

        const uint32_t tiles = walk.tiles();
        uint32_t id = blockIdx.x;                // of the tile that the streams walk towards
        typename Walk::Place ahead = walk.place(id), cur = ahead;
        uint32_t cur_id = id;
        SM sm;
        SN sn;
        sm.start(lane);
        sn.start(lane);
        sm.locate(walk.m(ahead), ahead.m0, wave);
        sn.locate(walk.n(ahead), ahead.n0, wave);
        auto advance_m = [&]() {                 // the M side comes to the end of a tile first (or together with the N side)
            sm.advance();
            if (sm.slabs_left != 0) return;
            id += gridDim.x;
            if (id < tiles) {
                ahead = walk.place(id);
                sm.locate(walk.m(ahead), ahead.m0, wave);
            } else sm.stop();
        };
        auto advance_n = [&]() {
            sn.advance();
            if (sn.slabs_left != 0) return;
            if (id < tiles) sn.locate(walk.n(ahead), ahead.n0, wave);
            else sn.stop();
        };
        // what steady state has requested before k-step 0 of slab 0; the first reads need the first slab only
        auto slab_m = [&](int from, int count) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < count) sm.request((from + q) & 3, lds_m, wave);
        };
        auto slab_n = [&](int from, int count) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < count) sn.request((from + q) & 3, lds_n, wave);
        };
        slab_m(TRM ? 1 : 3, 4);
        sm.advance();
        slab_n(TRN ? 1 : 3, 4);
        sn.advance();
        slab_m(TRM ? 1 : 3, TRM ? 2 : 4);
        if (!TRM) sm.advance();
        slab_n(TRN ? 1 : 3, TRN ? 2 : 4);
        if (!TRN) sn.advance();
        slab_m(3, 1);
        slab_n(3, 1);
        constexpr int kSecond = (TRM ? SM::I / 2 : SM::I) + (TRN ? SN::I / 2 : SN::I);
        constexpr int kBehind = SM::I + SN::I;   // requests of four k-steps
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kSecond) : "memory");

        Acc acc;
        bf16x8 a[2][FN], b[2][FM];
        uint32_t at_m = 0, at_n = 0;             // ring offsets of the slab that is read
        // read r of the fragments of a k-step: first what its first multiply needs
        auto read = [&](int r, int ks, int set) {
            const unsigned char *base_m = smem + at_m, *base_n = smem + SM::kRing + at_n;
            if (r == 0) b[set][0] = fm.read(base_m, ks, 0);
            else if (r == 1) a[set][0] = fn.read(base_n, ks, 0);
            else if (r < FM + 1) b[set][r - 1] = fm.read(base_m, ks, r - 1);
            else if (r < FM + FN) a[set][r - FM] = fn.read(base_n, ks, r - FM);
        };
        // k-step q: its multiplies, with the reads of the next one and the requests of q between them
        auto step = [&](int q) {
            const int set = q & 1;
            int r = 0;
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[set][j], b[set][i], acc[j][i], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    const int until = ((j * FM + i + 1) * (FM + FN) + FM * FN - 2) / (FM * FN - 1);
#pragma unroll
                    for (; r < until && r < FM + FN; ++r) read(r, (q + 1) & 3, set ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (j == 0 && i == FM - 1) {
                        sn.request(q, lds_n, wave);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (j == FN - 1 && i == FM - 1) {
                        sm.request(q, lds_m, wave);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
        };
        // The barrier before an odd k-step.  `landed`: everything requested up to the last epilogue has landed, which is
        // all that the first slab of a tile needs.
        bool landed = false;
        auto meet = [&]() {
            if (landed) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kBehind) : "memory");
        };

#pragma unroll
        for (int r = 0; r < FM + FN; ++r) read(r, 0, 0);
        for (;;) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;
            typename Walk::Held held;
            walk.begin(cur, held, wm * (32u * FM), wn * (32u * FN), fresh_lane());
            uint32_t left = __builtin_amdgcn_readfirstlane(max((cur.depth + kSlab - 1) / kSlab, kMinSlabs));
#pragma clang loop unroll(disable)
            do {
                step(0);
                if (TRM) advance_m();
                if (TRN) advance_n();
                meet();
                step(1);
                step(2);
                if (!TRM) advance_m();
                if (!TRN) advance_n();
                meet();
                landed = false;
                // from here on the next slab is read: of this tile or of the next (past the last tile: unused)
                at_m = at_m + SM::kBytes == (uint32_t)SM::kRing ? 0u : at_m + SM::kBytes;
                at_n = at_n + SN::kBytes == (uint32_t)SN::kRing ? 0u : at_n + SN::kBytes;
                step(3);
            } while (--left != 0);
            walk.finish(cur, acc, held, wm * (32u * FM), wn * (32u * FN), fresh_lane(), [&]() {
                if (!landed) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                landed = true;
            });
            cur_id += gridDim.x;
            if (cur_id >= tiles) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing may arrive in LDS after this workgroup
                break;
            }
            cur = ahead;         // crossed into by the request cursor at least one slab ago, and no further
        }
    }
};

// The same product with two workgroups per compute unit (M side major, N side tr): while one is in its epilogue, or waits,
// the other multiplies.  Half the LDS each: the M side has two slabs, the N side three half slabs of 32 k-rows.  Per
// slab two barriers, before k-steps 1 and 3.  After the first, the slab's first half of N has been read and its stage is
// requested into (second half of the next slab); after the other, its second half and the M slab (first half and M slab two
// ahead).  Requests have the three k-steps to the barrier that needs them.
// ONCE: the N side is requested non-temporally (weights that one row tile uses and that come from HBM).
template <int BM, int BN, int WM, int WN, bool ONCE = false>
struct TilePair {
    static constexpr int kWavesT = WM * WN, kThreads = 64 * kWavesT;
    static constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
    using SM = OperandStream<BM, false, kWavesT, 2>;
    using SN = OperandStream<BN, true, kWavesT, 3, kSlab / 2, ONCE>;
    static constexpr uint32_t kLds = SM::kRing + SN::kRing;
    static_assert(kLds <= 80 * 1024, "half the LDS of a compute unit");
    typedef f32x16 Acc[FN][FM];

    template <typename Walk>
    __device__ static void run(const Walk &walk, unsigned char *smem)
    {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t wm = wave / WN, wn = wave % WN;
        const uint32_t lds_m = lds_address(smem), lds_n = lds_m + SM::kRing;
        Fragments<BM, false, FM> fm;
        Fragments<BN, true, FN> fn;
        fm.init(wm * (32u * FM), lane);
        fn.init(wn * (32u * FN), lane);

        const uint32_t tiles = walk.tiles();
        uint32_t id = blockIdx.x;                // of the tile that the M stream walks towards
        typename Walk::Place ahead = walk.place(id), cur = ahead;
        uint32_t cur_id = id;
        SM sm;
        SN sn;
        sm.start(lane);
        sn.start(lane);
        sm.locate(walk.m(ahead), ahead.m0, wave);
        sn.locate(walk.n(ahead), ahead.n0, wave);
        // Crossed into right before the first request of the next tile, the M side first (k-step 3 of the last but one slab).
        auto cross_m = [&]() {
            if (sm.slabs_left != 0) return;
            id += gridDim.x;
            if (id < tiles) {
                ahead = walk.place(id);
                sm.locate(walk.m(ahead), ahead.m0, wave);
            } else sm.stop();
        };
        auto cross_n = [&]() {
            if (sn.slabs_left != 0) return;
            if (id < tiles) sn.locate(walk.n(ahead), ahead.n0, wave);
            else sn.stop();
        };
        auto fetch_m = [&]() {
#pragma unroll
            for (int i = 0; i < SM::I; ++i) sm.fetch(i, lds_m, wave);
            sm.advance();
        };
        auto fetch_n = [&]() {
#pragma unroll
            for (int i = 0; i < SN::I; ++i) sn.fetch(i, lds_n, wave);
            sn.advance();
        };
        // what steady state has requested before k-step 0 of slab 0, of which the first reads need the first two
        fetch_m();
        fetch_n();
        fetch_n();
        fetch_m();
        fetch_n();
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(SM::I + 2 * SN::I) : "memory");

        Acc acc;
        bf16x8 a[2][FN], b[2][FM];
        uint32_t at_m = 0, at_n = 0;             // ring offsets of what is read
        auto read = [&](int r, int ks, int set) {
            const unsigned char *base_m = smem + at_m, *base_n = smem + SM::kRing + at_n;
            if (r == 0) b[set][0] = fm.read(base_m, ks, 0);
            else if (r == 1) a[set][0] = fn.read(base_n, ks & 1, 0);
            else if (r < FM + 1) b[set][r - 1] = fm.read(base_m, ks, r - 1);
            else if (r < FM + FN) a[set][r - FM] = fn.read(base_n, ks & 1, r - FM);
        };
        // k-step q: its multiplies, with the reads of the next one and the requests of q between them
        auto step = [&](int q) {
            const int set = q & 1;
            int r = 0, f = 0;
            const int requests = q == 1 ? SN::I : q == 3 ? SN::I + SM::I : 0;
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[set][j], b[set][i], acc[j][i], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    const int n = j * FM + i + 1;
                    const int until = (n * (FM + FN) + FM * FN - 2) / (FM * FN - 1);
#pragma unroll
                    for (; r < until && r < FM + FN; ++r) read(r, (q + 1) & 3, set ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                    const int upto = n * requests / (FM * FN);
#pragma unroll
                    for (; f < upto; ++f) {
                        if (q == 3 && f < SM::I) sm.fetch(f, lds_m, wave);
                        else sn.fetch(f - (q == 3 ? SM::I : 0), lds_n, wave);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            if (q == 3) sm.advance();
            if (q & 1) sn.advance();
        };
        bool landed = false;                     // everything requested up to the last epilogue
        auto next_n = [&]() { at_n = at_n + SN::kBytes == (uint32_t)SN::kRing ? 0u : at_n + SN::kBytes; };

#pragma unroll
        for (int r = 0; r < FM + FN; ++r) read(r, 0, 0);
        for (;;) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;
            uint32_t left = __builtin_amdgcn_readfirstlane(max((cur.depth + kSlab - 1) / kSlab, kMinSlabs));
#pragma clang loop unroll(disable)
            do {
                step(0);
                if (landed) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(SM::I + SN::I) : "memory");
                next_n();
                step(1);
                step(2);
                if (landed) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(SN::I) : "memory");
                landed = false;
                cross_m();
                cross_n();
                next_n();
                at_m = at_m + SM::kBytes == (uint32_t)SM::kRing ? 0u : at_m + SM::kBytes;
                step(3);
            } while (--left != 0);
            walk.finish(cur, acc, typename Walk::Held{}, wm * (32u * FM), wn * (32u * FN), fresh_lane(), [&]() {
                if (!landed) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                landed = true;
            });
            cur_id += gridDim.x;
            if (cur_id >= tiles) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing may arrive in LDS after this workgroup
                break;
            }
            cur = ahead;
        }
    }
};

// The same tiles for launches that are bound by the weight stream (few rows per job): what counts is bytes in flight per
// compute unit, so LDS is one ring of D whole slabs per operand, D - 1 of them on their way, and the walk across
// tiles keeps it full through the epilogues.  One barrier per slab: after it slab s has landed for everyone
// and everyone has left the stage of slab s - 1, which is requested into at once.  HALVES: two sums per output, over the first and
// over the second two k-steps of every slab, added at the end of a tile.
template <int BM, int BN, int WM, int WN, bool TRN, int D, bool HALVES = false>
struct TileStream {
    static constexpr int kWavesT = WM * WN, kThreads = 64 * kWavesT;
    static constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
    using SM = OperandStream<BM, false, kWavesT, D>;
    using SN = OperandStream<BN, TRN, kWavesT, D>;
    static constexpr uint32_t kLds = SM::kRing + SN::kRing;
    static constexpr int kBehind = (D - 2) * (SM::I + SN::I);
    static_assert(kLds <= 160 * 1024 && kBehind <= 63, "LDS of a compute unit, largest count of s_waitcnt");
    typedef f32x16 Acc[FN][FM];

    template <typename Walk>
    __device__ static void run(const Walk &walk, unsigned char *smem)
    {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t wm = wave / WN, wn = wave % WN;
        const uint32_t lds_m = lds_address(smem), lds_n = lds_m + SM::kRing;
        Fragments<BM, false, FM> fm;
        Fragments<BN, TRN, FN> fn;
        fm.init(wm * (32u * FM), lane);
        fn.init(wn * (32u * FN), lane);
        const uint32_t tiles = walk.tiles();
        uint32_t id = blockIdx.x, cur_id = id;
        typename Walk::Place ahead = walk.place(id), cur = ahead;
        SM sm;
        SN sn;
        sm.start(lane);
        sn.start(lane);
        sm.locate(walk.m(ahead), ahead.m0, wave);
        sn.locate(walk.n(ahead), ahead.n0, wave);
        // part of four of the requests of the slab under the cursors; the last one moves on
        auto request = [&](int part) {
#pragma unroll
            for (int i = 0; i < SN::I + SM::I; ++i) {
                if (i * 4 / (SN::I + SM::I) != part) continue;
                if (i < SN::I) sn.fetch(i, lds_n, wave);
                else sm.fetch(i - SN::I, lds_m, wave);
            }
            if (part != 3) return;
            sm.advance();
            sn.advance();
            if (sm.slabs_left != 0) return;
            id += gridDim.x;
            if (id < tiles) {
                ahead = walk.place(id);
                sm.locate(walk.m(ahead), ahead.m0, wave);
                sn.locate(walk.n(ahead), ahead.n0, wave);
            } else {
                sm.stop();
                sn.stop();
            }
        };
#pragma clang loop unroll(disable)
        for (int d = 0; d < D - 1; ++d)
#pragma unroll
            for (int part = 0; part < 4; ++part) request(part);

        constexpr int kSums = HALVES ? 2 : 1;
        Acc acc[kSums];
        uint32_t stage = 0;
        for (;;) {
#pragma unroll
            for (int c = 0; c < kSums; ++c)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[c][j][i][r] = 0.f;
            uint32_t left = __builtin_amdgcn_readfirstlane(max((cur.depth + kSlab - 1) / kSlab, kMinSlabs));
#pragma clang loop unroll(disable)
            do {
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kBehind) : "memory");
                const unsigned char *base_m = smem + stage * SM::kBytes, *base_n = smem + SM::kRing + stage * SN::kBytes;
                bf16x8 a[4][FN], b[4][FM];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
                    for (int i = 0; i < FM; ++i) b[ks][i] = fm.read(base_m, ks, i);
#pragma unroll
                    for (int j = 0; j < FN; ++j) a[ks][j] = fn.read(base_n, ks, j);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    request(ks);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int i = 0; i < FM; ++i)
                            acc[ks * kSums / 4][j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][j], b[ks][i], acc[ks * kSums / 4][j][i], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                stage = stage + 1 == (uint32_t)D ? 0u : stage + 1;
            } while (--left != 0);
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int r = 0; HALVES && r < 16; ++r) acc[0][j][i][r] += acc[kSums - 1][j][i][r];
            walk.finish(cur, acc[0], typename Walk::Held{}, wm * (32u * FM), wn * (32u * FN), fresh_lane(), []() {});
            cur_id += gridDim.x;
            if (cur_id >= tiles) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing may arrive in LDS after this workgroup
                break;
            }
            cur = walk.place(cur_id);          // the requests may be more than one tile ahead
        }
    }
};

// ---- a wavefront's accumulators in line order -------------------------------------------------------------
// Accumulator register r of a 32 x 32 block in lane l: row l % 32, column 8 (r / 4) + 4 (l / 32) + r % 4.
// Each exchange below swaps one bit of the register number (a column bit) with one bit of the lane (a row bit,
// or for the first the column bit 4 of l / 32), until eight lanes together hold a 128-byte line.
__device__ inline void swap_halves(uint32_t &x, uint32_t &y)      // lane bit 5
{
    const auto s = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = s[0];
    y = s[1];
}
__device__ inline void swap_rows(uint32_t &x, uint32_t &y)        // lane bit 4
{
    const auto s = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = s[0];
    y = s[1];
}
__device__ inline void swap_eights(uint32_t &x, uint32_t &y)      // lane bit 3
{
    const uint32_t x0 = x;
    x = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)y, 0x128 /* row_ror:8 */, 0xf, 0xc, false);
    y = (uint32_t)__builtin_amdgcn_update_dpp((int)y, (int)x0, 0x128, 0xf, 0x3, false);
}

// Two 32 x 32 blocks side by side (64 columns) as bf16: out[a][b] is row 16 a + 8 b + l % 8, columns
// line_column_bf16(l) .. + 7.
__device__ inline void to_lines_bf16(const float (&v)[2][16], u32x4 (&out)[2][2])
{
    uint32_t p[2][4][2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int d = 0; d < 2; ++d) p[j][q][d] = bf16_pack(v[j][4 * q + 2 * d], v[j][4 * q + 2 * d + 1]);
#pragma unroll
    for (int d = 0; d < 2; ++d) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            // register bit 3 of the column <-> lane bit 5 (bit 2 of the column): p[j][2 h + x]: column bit 4 = h, bit 2 = x
            swap_halves(p[j][0][d], p[j][1][d]);
            swap_halves(p[j][2][d], p[j][3][d]);
            // column bit 4 <-> lane bit 4 (row bit 4)
            swap_rows(p[j][0][d], p[j][2][d]);
            swap_rows(p[j][1][d], p[j][3][d]);
        }
        // column bit 5 (j) <-> lane bit 3 (row bit 3)
#pragma unroll
        for (int q = 0; q < 4; ++q) swap_eights(p[0][q][d], p[1][q][d]);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) out[a][b] = u32x4{p[b][2 * a][0], p[b][2 * a][1], p[b][2 * a + 1][0], p[b][2 * a + 1][1]};
}
__device__ inline uint32_t line_column_bf16(int lane) { return 32u * ((lane >> 3) & 1u) + 16u * ((lane >> 4) & 1u) + 8u * (lane >> 5); }

// One 32 x 32 block as bf16, half lines: out[a] is row 16 a + l % 16, columns half_line_column_bf16(l) .. + 7.
__device__ inline void to_half_lines_bf16(const float (&v)[16], u32x4 (&out)[2])
{
    uint32_t p[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int d = 0; d < 2; ++d) p[q][d] = bf16_pack(v[4 * q + 2 * d], v[4 * q + 2 * d + 1]);
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        swap_halves(p[0][d], p[1][d]);           // as the first two exchanges of to_lines_bf16
        swap_halves(p[2][d], p[3][d]);
        swap_rows(p[0][d], p[2][d]);
        swap_rows(p[1][d], p[3][d]);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) out[a] = u32x4{p[2 * a][0], p[2 * a][1], p[2 * a + 1][0], p[2 * a + 1][1]};
}
__device__ inline uint32_t half_line_column_bf16(int lane) { return 16u * ((lane >> 4) & 1u) + 8u * (lane >> 5); }

// One 32 x 32 block as float: out[a][b] is row 16 a + 8 b + l % 8, columns line_column_f32(l) .. + 3.
__device__ inline void to_lines_f32(const float (&v)[16], f32x4 (&out)[2][2])
{
    uint32_t p[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) p[q][e] = __builtin_bit_cast(uint32_t, v[4 * q + e]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        swap_rows(p[0][e], p[1][e]);             // column bit 3 <-> row bit 4
        swap_rows(p[2][e], p[3][e]);
        swap_eights(p[0][e], p[2][e]);           // column bit 4 <-> row bit 3
        swap_eights(p[1][e], p[3][e]);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) out[a][b][e] = __builtin_bit_cast(float, p[2 * b + a][e]);
}
__device__ inline uint32_t line_column_f32(int lane) { return 16u * ((lane >> 3) & 1u) + 8u * ((lane >> 4) & 1u) + 4u * (lane >> 5); }

// A tile's offsets stay below 2 GB (the descriptor's range): 256 rows of K values, 64 rows of N, a strip of K x 128.
constexpr uint32_t kTiledMaxWidth = 1u << 22;

// Workgroups of a launch with one resident workgroup per compute unit; a multiple of 8, so that the workgroups of an
// XCD keep to that XCD's range of tiles.
inline uint32_t resident_grid()
{
    static uint32_t cached = 0;
    if (cached) return cached;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8)
        cus = 256;
    cached = (uint32_t)cus & ~7u;
    return cached;
}

}  // namespace salus
