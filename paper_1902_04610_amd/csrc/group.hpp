// Pieces shared by the grouped dense kernels: the by-value argument block, the
// epilogue arithmetic and the workgroup -> (job, tile) lookup.
#pragma once
#include "device.hpp"
#include "wave.hpp"

namespace salus {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct GroupArgs {
    uint32_t n;
    uint32_t tiles;      // all tiles of the launch
    uint32_t past_l2;    // kernels whose workgroups loop over tiles: float outputs whose rows begin on a line are stored past L2
    uint32_t pad;
    uint32_t first[kMaxProblems];      // first tile of problem i; kNoTile from n on
    Problem p[kMaxProblems];
};
constexpr uint32_t kNoTile = ~0u;
static_assert(sizeof(GroupArgs) <= 4096, "kernel arguments are limited to 4 KB");
struct InOrderArgs : GroupArgs {};      // names the variant of a kernel that adds every output's products in order of k

// The same for launches of few problems, whose time is the host's: a launch with 3.3 KB of arguments takes it 0.4 us longer than one with
// 0.4 KB (3.7 us).  2 float jobs x 8 rows, 256 - 256 - 256, two launches: 9.2 us a round, 8.5 so.
constexpr uint32_t kFewProblems = 8;
struct FewArgs {
    uint32_t n, tiles, past_l2, pad;
    uint32_t first[kFewProblems];
    Problem p[kFewProblems];
};

// Fills in a launch of at most as many problems as Args holds, whose i-th has tiles(problem) tiles; returns how many there are in all.
template <typename Args, typename P, typename Tiles>
inline uint64_t fill_group(Args &a, const P *p, uint32_t n, Tiles tiles)
{
    uint64_t total = 0;
    a.n = n;
    for (uint32_t i = 0; i < n; ++i) {
        a.p[i] = p[i];
        a.first[i] = (uint32_t)total;
        total += tiles(p[i]);
    }
    for (uint32_t i = n; i < sizeof(a.first) / sizeof(a.first[0]); ++i) a.first[i] = kNoTile;
    a.tiles = (uint32_t)total;
    return total;
}

constexpr int kGemmThreads = 256;
constexpr int kWaves = 4;

// bf16 kernels: GELU(z) = z / 2 + |z| (1/2 - Q(|z|)) with the upper tail Q(x) = erfc(x / sqrt 2) / 2 = 2^p(x), p the
// polynomial of degree 6 that minimizes the largest |x (2^p - Q)| over [0, 5.5] (fitted by linear programming; 9.8e-8 with the coefficients in float),
// evaluated up to 9, from where on Q is below 2^-62 and 1/2 - Q is 1/2.  Fourteen operations, counting the exponential
// (v_exp_f32) as four: the epilogues of wide layers are bound by them, and where the power limit sets the clock they cost
// what multiplies could use (16 jobs x 4096 rows, 1024 - 4096 - 1024 - 1024: 1186 us, 1264 with the rational
// approximation of erfc before it).  In float arithmetic over [-40, 40]: |error| of the result below 4e-7 (7.6e-7).  The error is *absolute* in Q,
// so for z < -3.5, where Q itself falls below 5e-4, the relative error of a single output grows; such outputs are below
// 1e-3 in magnitude and only decide a comparison when a whole matrix consists of them.  Infinities give what the sum
// of z / 2 and |z| / 2 gives, a NaN stays a NaN.
__device__ inline float gelu_fast(float z)
{
    const float x = fabsf(z), c = __builtin_amdgcn_fmed3f(x, 0.0f, 9.0f);
    float p = fmaf(2.90425268758554e-05f, c, -0.0007323235622607172f);
    p = fmaf(p, c, 0.007953787222504616f);
    p = fmaf(p, c, -0.05320511385798454f);
    p = fmaf(p, c, -0.45893481373786926f);
    p = fmaf(p, c, -1.1511449813842773f);
    p = fmaf(p, c, -0.9999991059303284f);
    const float q = __builtin_amdgcn_exp2f(p);
    return fmaf(x, 0.5f - q, 0.5f * z);
}

__device__ inline float activate(float z, uint32_t act)
{
    if (act == 1) return fmaxf(z, 0.0f);
    if (act == 2) return gelu_fast(z);
    return z;
}

// float kernels: the bound is relative (1e-5 of the largest output), so GELU is
// 0.5 z erfc(-z / sqrt 2) with the library's erfc, accurate to a few ulp in the
// negative tail as well.  These kernels are latency-bound; the cost does not show.
__device__ inline float activate_f32(float z, uint32_t act)
{
    if (act == 1) return fmaxf(z, 0.0f);
    if (act == 2) return 0.5f * z * erfcf(-0.70710678118654752440f * z);
    return z;
}

// float -> bf16 bits, round to nearest, ties to even (v_cvt_pk_bf16_f32).
__device__ inline uint32_t bf16_bits(float f)
{
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// two floats -> two bf16 in one dword (a in the low half), one instruction
__device__ inline uint32_t bf16_pack(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// Workgroups are dealt round-robin to the 8 XCDs (each with its own L2); map
// the hardware index to a logical one so that every XCD works on a contiguous
// range of tiles - the tiles of one job share its activations in one L2.
__device__ inline uint32_t xcd_remap(uint32_t b, uint32_t total)
{
    const uint32_t x = b & 7u, slot = b >> 3;
    const uint32_t q = total >> 3, r = total & 7u;
    return x * q + (x < r ? x : r) + slot;
}

// Which problem of a launch the tile `id` belongs to: copied to `owner`; returns the tile's number among that problem's.
// Nothing can begin before this answer, so it is one trip to memory: lane i loads problem i and its first tile, a ballot
// finds the last one that begins at or before `id`, and that lane is read out.  0.6 us from a workgroup's start; scanning
// tile counts and then reading the problem by its number, three dependent trips, took 1.6: one request against a 1024 -
// 4096 - 1024 - 1024 model, three launches, 26.1 / 24.1 us, 64 such models 174.5 / 172.5.
template <typename P, uint32_t NP>
__device__ inline uint32_t find_owner(const uint32_t (&first)[NP], const P (&p)[NP], uint32_t id, P &owner)
{
    constexpr int kWords = sizeof(P) / 4;
    struct Words { uint32_t w[kWords]; };
    const uint32_t lane = threadIdx.x & 63, at = NP == 64 ? lane : min(lane, NP - 1);
    const uint32_t from = first[at];
    const Words mine = __builtin_bit_cast(Words, p[at]);
    const int g = __builtin_amdgcn_readfirstlane(wave_find_range(from, id, lane < NP));
    Words words;
#pragma unroll
    for (int i = 0; i < kWords; ++i) words.w[i] = __builtin_amdgcn_readlane(mine.w[i], g);
    owner = __builtin_bit_cast(P, words);
    return id - __builtin_amdgcn_readlane(from, g);
}

struct Tile {
    uint32_t m0, n0;
};

// Which (job, row tile, column tile) this workgroup owns, and that job's problem.
template <int TM, int TN, typename Args>
__device__ inline Tile find_tile(const Args &a, Problem &p)
{
    const uint32_t t = find_owner(a.first, a.p, xcd_remap(blockIdx.x, a.tiles), p), rt = (p.M + TM - 1) / TM;
    return {(t % rt) * TM, (t / rt) * TN};      // row tiles of one column tile are neighbours: they share W
}

}  // namespace salus
