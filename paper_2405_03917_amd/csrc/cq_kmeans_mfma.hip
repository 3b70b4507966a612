// One Lloyd iteration of the centroid learning (cq_kmeans.hip says what it computes) for groups of
// 256 centroids, with the matrix cores as a FILTER and the fp32 direct form as the judge, and the
// cluster sums accumulated while the token is in registers.
//
// The assignment is defined as the argmin of the direct form D_j = sum_i (x_i - c_i)^2 in fp32
// (lowest index among equals).  In exact arithmetic argmin_j D_j = argmax_j s_j with
// s_j = x . c_j - |c_j|^2 / 2.  One v_mfma_f32_32x32x16_f16 scores 32 tokens against 32 centroids:
// its K dimension carries the c channels twice, against the high and the low fp16 part of the
// fp32 centroid (22 bits), and -|c_j|^2 / 2 enters through the accumulator.  Each lane keeps the two
// largest maxima of 8 scores it sees (the number of the eight packed into the four lowest mantissa
// bits: 13 vector instructions per 16 scores).  The eight centroids of the winner are then
// compared in the direct form; if the winner's maximum beats the runner-up's by more than the
// bound below, no other centroid can have a smaller direct-form distance, and the choice IS the
// direct form's argmin, bit for bit.  Otherwise the token is re-done against all centroids in
// the direct form.
//
// Scaling.  Tokens and centroids are multiplied by a power of two 2^s that brings the largest
// |c|^2 into [2^12, 2^14): both then sit inside fp16's normal range where it matters.  (s < 0 can
// push a token's channel into the subnormals: an absolute error below 2^-24, against a unit of
// the bound of 2^-9 or more.)  Groups whose centroids are all (nearly) zero and tokens more
// than 256 times longer than the longest centroid go to the direct form whole.
//
// Bound.  M = |x'| |c'| + |c'|^2 / 2 (scaled) of the centroid in question, in units of 2^-20 M.  A
// score: low part of the centroid 0.25, |c|^2 in fp32 0.5, the matrix core's sum of 16 exact
// products and the accumulator 2.3 (at most 2^-23 M each and for the rounding): 3.05, twice for
// a difference, and 1.9 for the packed bits (both are cut): 8.  The direct form errs by at most
// (c + 2) 2^-24 of each distance, distances are at most |x'|^2 + 2 M, half of it counts for a
// score: 1.25 M + 0.625 |x'|^2.  The test uses 11 M + 0.75 |x'|^2.  Only centroids that could be as
// near as the winner (direct-form distance d), or whose score came out as high as its, matter:
// |c'| <= |x'| + sqrt(d') for the first; for the second d' + 4 x 8 2^-20 M_max in the root, whose
// share is at most 0.0068 sqrt(|x'|^2 + |c'|max^2) (`slack`).  That norm, `reach`, goes into M: with
// M_max there a group with a few long centroids sent three times as many tokens to the re-do.
//
// Equal centroids (more centroids than distinct points, dead channels, coarse values) would tie for every token
// near them; all but the first of them leave the scan, found by a hash table when the group's centroids are read.
// 4096 tokens of 40 distinct points, 128 groups of 8 channels, per iteration: 76 us in the direct search of all, 419
// when every tie was re-done, 60 now; half of the channels dead: 115, 434, 51.
// (A table of 4096 slots misses fewer of them, 617 -> 532 us for 10 iterations of 4096 weighted tokens of integers in
// 256 groups of 4, but its clearing costs calls of 300 to 1500 tokens, groups of 2, 3 to 6 %.)
//
// Skipping.  In a fit of many iterations most tokens keep their centroid.  When a token has been looked at, its
// distance d to its centroid a and a lower bound b of its distance to every other are known (the runner-up's score
// and the winner's eight, less the bound above for the longest centroid).  Until a has moved by D_a and no centroid by
// more than D in all, with D_a + D < b - d, a is still the nearest (Hamerly, "Making k-means even faster", 2010).
// So each token keeps one number, its threshold t = (b - d) + D_a + D at that time, and is skipped while
// t > D_a + D; the sums of the clusters stay from one iteration to the next, and only tokens that change cluster are
// moved (integers: the same sums, and the same centroids, whatever the order).  The choice must be that of the
// direct form in fp32, so nothing is left to rounding: lengths carry 2^-18 of themselves as a margin (the direct
// form's error is 3 x 2^-22 of the squares), moves are rounded up, thresholds down (fp16, scaled; at most 65504);
// near ties and every token of a group with equal centroids (which a twin that stays behind could win) get 0 and are
// looked at again.
// A wavefront lists its tokens that are not skipped and takes 64 of the list at a time.  Such an iteration costs
// 1.2 to 1.3 times a plain one when it skips nothing, and 0.15 when it skips everything; of 100 iterations over the
// calibration tokens (32768, groups of 8) 0.4 of the tokens are looked at, 0.8 in the first ten.  An iteration that moves
// no centroid at all is the same as every later one: the group is done, in this launch and in those behind it.  (Without
// that, groups of more centroids than distinct points, all of whose tokens are looked at again, took longer than plain
// iterations: 100 iterations of 32768 tokens of 40 points, 512 groups 57.2 ms plain, 68.6, and 6.4 now; of 4000 tokens of
// integers, 2048 groups of 2, 11.7, 14.3 and 1.4.)
// All iterations, plain -> now (starts from k-means++): 32768 tokens, 512 groups, 100 iterations 32.9 -> 20.8 ms, weighted
// 41.3 -> 18.7; 6000 tokens 6.6 -> 2.2; 30 iterations 1.06 to 1.7 times as fast; 20 iterations, were they to skip, 0.88 to 1.13
// times (hence kStateIterations, kPlainIterations).  What stays slower are unweighted starts far from the tokens (random
// tokens stretched up to six times and shifted), 8 channels: 30 iterations 0.85 to 0.96, 60 0.89 to 1.03, 100 from 1.00 on.
// Weighted fits of few tokens (below about 12000 of 8 channels) have no room for the sums in their scratch and run plain.
// A group's only workgroup runs many iterations in one launch: 100 launches waited for their busiest
// group each (26.3 against 30.3 ms).
//
// What bounds it: the vector ALU (a plain iteration 545 instructions per 64 tokens and group: 208 in the scan, 150 in
// the winner's eight, the rest merge, bound, sums and re-dos; the direct search took 2 c + 3 per
// token and centroid).  The group's centroids sit in registers as matrix operands (32 registers)
// with the norms in accumulator layout (128; half of them read from LDS where tokens are skipped): two wavefronts per
// SIMD and no other LDS reads in the scan.  32768 tokens, 512 groups of 8 channels: 1.36 + 0.30 ms per iteration in two kernels ->
// 0.31 ms (maxima over quads instead of eights: 17 instructions per 16 scores in the scan for 4
// fewer distances per token, slower by the count).
//
// This file is compiled with -fno-honor-nans (bare v_max3_f32 / v_med3_f32).  Non-finite input
// gives unspecified assignments, always in range.
#include "cq_kmeans_common.hpp"
#include "cq_kmeans_mfma.hpp"

namespace cq {
namespace {

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kLloydWaves = 4;
constexpr int kK = 256;                 // centroids per group
constexpr int kNBlk = kK / 32;
constexpr int kHashSlots = 1024;        // for finding equal centroids
constexpr int kStateIterations = 30;    // a fit of at least as many iterations skips tokens, ...
constexpr int kPlainIterations = 10;    // ... from this iteration on
constexpr int kLaunchIterations = 128;  // one launch takes at most so many iterations, ...
constexpr int kLaunchTokens = 1 << 22;  // ... and so many tokens of a group times iterations (see launch_lloyd)
static_assert(kStateIterations >= kPlainIterations + 2, "one iteration fills the state, at least one uses it");

template <int CTRL>
__device__ __forceinline__ unsigned dpp_mov(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}
// minimum / maximum over the 64 lanes (all active), wavefront-uniform
template <bool MAX>
__device__ __forceinline__ unsigned wave_extreme_u32(unsigned v)
{
    auto pick = [](unsigned a, unsigned b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); };
    v = pick(v, dpp_mov<0xB1>(v));      // quad_perm [1,0,3,2]
    v = pick(v, dpp_mov<0x4E>(v));      // quad_perm [2,3,0,1]
    v = pick(v, dpp_mov<0x141>(v));     // row_half_mirror
    v = pick(v, dpp_mov<0x140>(v));     // row_mirror
    const unsigned a = pick((unsigned)__builtin_amdgcn_readlane((int)v, 0), (unsigned)__builtin_amdgcn_readlane((int)v, 16));
    const unsigned b = pick((unsigned)__builtin_amdgcn_readlane((int)v, 32), (unsigned)__builtin_amdgcn_readlane((int)v, 48));
    return pick(a, b);
}

// The x_i of a token's group slice as the words they are stored in.
template <int C>
__device__ __forceinline__ void load_words(const uint16_t* p, unsigned (&w)[C / 2])
{
    if constexpr (C == 8) {
        const uint4 v = *reinterpret_cast<const uint4*>(p);
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else if constexpr (C == 4) {
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        w[0] = v.x; w[1] = v.y;
    } else {
        w[0] = *reinterpret_cast<const unsigned*>(p);
    }
}
template <int C>
__device__ __forceinline__ void widen_words(const unsigned (&w)[C / 2], float (&v)[C])
{
#pragma unroll
    for (int i = 0; i < C / 2; ++i) {
        const half2_t h = __builtin_bit_cast(half2_t, w[i]);
        v[2 * i] = (float)h.x;
        v[2 * i + 1] = (float)h.y;
    }
}

// 1.5 2^23: adding an integer below 2^22 in size leaves it in the low mantissa bits
constexpr float kMagic = 12582912.f;
constexpr unsigned kMagicBits = 0x4b400000u;
// sum of x 2^24 of `count` tokens from the sum of their bit patterns
__device__ __forceinline__ long long plain_sum(unsigned long long s, unsigned long long count)
{
    return (long long)(s - count * (((unsigned long long)kMagicBits << 20) + kMagicBits));
}

template <int C>
struct Operand {
    using type = half4_t;
};
template <>
struct Operand<8> {
    using type = half8_t;
};

// Sums of one cluster: unweighted C sums of x 2^24 and the count; weighted C pairs (high, low) and
// the weight.  (C odd strides in 8-byte words: neighbouring clusters start in different banks.)
template <int C, bool W>
constexpr int kSumWords = (W ? 2 * C : C) + 1;

// What the iterations of one fit hand on from each to the next where tokens may be skipped ("Skipping" above).
// Per group g: sums [256][kSumWords] of the present assignment; travel, kTravelWords floats: how far each centroid
// has moved since the first iteration, the sum of the longest moves, the scale of lengths of the first
// iteration, and whether an iteration has moved no centroid; per token its threshold (fp16) and its cluster.
constexpr int kTravelWords = kK + 4;
struct LloydState {
    unsigned long long* sums;
    float* travel;
    unsigned* arrived;                  // workgroups of the group that are done (several splits per group)
    uint16_t* threshold;                // [group][n_pad]
    uint8_t* own;                       // [group][n_pad]
    int n_pad;
};
enum LloydMode { kPlain, kFirst, kNext };       // without state; fills it; uses it

constexpr int kScanTokens = 8;          // tokens whose thresholds a lane looks at together (16 bytes)
constexpr int kListTokens = 64 * kScanTokens + 64;

// One workgroup: tokens [split * tokens_per_split, ...) of one group.  One split per group: the new
// centroids are written at once; else the sums go to `partials` [group][split][256][kSumWords], or (with state) are
// added to the group's, and the last of its workgroups writes the centroids.
template <int C, bool W, int MODE>
__global__ __launch_bounds__(kLloydWaves * 64, 2) void kmeans_lloyd_kernel(const uint16_t* __restrict__ xg_all,
                                                                        const uint32_t* __restrict__ wq_all,
                                                                        float* cent_all, uint16_t* __restrict__ assign_all,
                                                                        unsigned long long* __restrict__ partials, LloydState state,
                                                                        int n, int tokens_per_split, int iterations)
{
    using vec_t = typename Operand<C>::type;
    constexpr int QS = 4 * C + 4;                       // floats per four centroids (16 bytes of padding: lanes that read
                                                        // different fours spread over the banks)
    constexpr int SW = kSumWords<C, W>;
    constexpr float LOWEST = -3.0e38f;
    __shared__ __attribute__((aligned(16))) float cs[kK / 4 * QS];
    __shared__ __attribute__((aligned(16))) float norms[kK];
    __shared__ unsigned c2w[kLloydWaves];
    __shared__ unsigned first_of[kHashSlots];
    __shared__ unsigned kept[kLloydWaves];
    __shared__ unsigned long long sums[kK * SW];
    __shared__ float need[MODE == kNext ? kK : 1];      // a token of cluster k is skipped if its threshold is above need[k]
    __shared__ unsigned long long changed[MODE == kNext ? kLloydWaves : 1][MODE == kNext ? 128 : 1];    // token, old cluster, new cluster
    __shared__ unsigned list[MODE == kNext ? kLloydWaves : 1][MODE == kNext ? kListTokens : 1];     // tokens to look at, cluster << 24

    int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.y, split = blockIdx.x;
    const uint16_t* xg = xg_all + (size_t)g * n * C;
    const uint32_t* wq = W ? wq_all + (size_t)g * n : nullptr;
    float* cent = cent_all + (size_t)g * kK * C;
    float* travel = MODE == kPlain ? nullptr : state.travel + (size_t)g * kTravelWords;
    uint16_t* threshold = MODE == kPlain ? nullptr : state.threshold + (size_t)g * state.n_pad;
    uint8_t* own_cluster = MODE == kPlain ? nullptr : state.own + (size_t)g * state.n_pad;
    float travelled = MODE == kNext ? travel[tid] : 0.f, longest = MODE == kNext ? travel[kK] : 0.f;
    const float f0 = MODE == kNext ? travel[kK + 1] : 0.f;
    unsigned long long* all_sums = MODE == kPlain ? nullptr : state.sums + (size_t)g * (kK * SW);
    auto write_assignment = [&](int from, int to) {
        for (int i = from + tid; i < to; i += kLloydWaves * 64) assign_all[(size_t)g * n + i] = own_cluster[i];
    };
    if (MODE == kNext && travel[kK + 2] != 0.f) {           // an earlier launch moved no centroid
        if (assign_all) write_assignment(split * tokens_per_split, min((split + 1) * tokens_per_split, n));
        return;
    }
    const bool alone = gridDim.x == 1;                  // the group's only workgroup
    for (int i = tid; i < kK * SW; i += kLloydWaves * 64) sums[i] = MODE == kNext && alone ? all_sums[i] : 0ull;

    // A group's only workgroup takes several iterations (groups end when they are done: the launch waits once for the
    // busiest of them); else `iterations` is 1.
#pragma unroll 1
    for (int it = 0;; ++it) {
    // (opaque: addresses that follow from them would be kept in registers through all iterations)
    if constexpr (MODE == kNext) asm volatile("" : "+v"(tid), "+v"(lane));
    const bool last_iteration = it + 1 >= iterations;
    uint16_t* assign_now = last_iteration ? assign_all : nullptr;

    // ---- the group's centroids: fp32 in LDS, scale, norms, matrix operands
    static_assert(kLloydWaves * 64 == kK, "one centroid per thread");
    float n2 = 0.f, own[C];
    unsigned hash = 0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        own[i] = it == 0 ? cent[(size_t)tid * C + i] : cs[(tid >> 2) * QS + (tid & 3) * C + i];
        n2 = __builtin_fmaf(own[i], own[i], n2);
        cs[(tid >> 2) * QS + (tid & 3) * C + i] = own[i];
        hash = (hash ^ __float_as_uint(own[i] + 0.f)) * 0x9e3779b1u;        // (zeros of both signs are equal)
        hash ^= hash >> 15;
    }
    hash = (hash * 0x85ebca6bu) / (0xffffffffu / kHashSlots + 1u);
    for (int i = tid; i < kHashSlots; i += kLloydWaves * 64) first_of[i] = ~0u;
    const unsigned wmax = wave_extreme_u32<true>(__float_as_uint(n2));
    if (lane == 0) c2w[wave] = wmax;
    if constexpr (MODE == kNext) need[tid] = (travelled + longest) * (1.f + 0x1p-22f);
    __syncthreads();
    unsigned c2bits = 0;
#pragma unroll
    for (int w = 0; w < kLloydWaves; ++w) c2bits = c2w[w] > c2bits ? c2w[w] : c2bits;
    atomicMin(&first_of[hash], (unsigned)tid);
    c2bits = (unsigned)__builtin_amdgcn_readfirstlane((int)c2bits);
    const int e = (int)((c2bits >> 23) & 0xffu) - 127;
    int s = (13 - e) >> 1;
    const bool extreme = s > 30 || s < -13;             // (nearly) all-zero centroids (or not finite)
    s = s > 30 ? 30 : (s < -13 ? -13 : s);
    const int s1 = s >> 1, s2 = s - s1;
    const unsigned m1b = (unsigned)(15 + s1) << 10, m2b = (unsigned)(15 + s2) << 10;      // fp16 2^s1, 2^s2
    const half2_t m1 = __builtin_bit_cast(half2_t, m1b | (m1b << 16)), m2 = __builtin_bit_cast(half2_t, m2b | (m2b << 16));
    const float f1 = __uint_as_float((unsigned)(127 + s) << 23), f2 = f1 * f1;
    const float c2s = __uint_as_float(c2bits) * f2;     // the largest |c'|^2
    __syncthreads();
    // A centroid equal to an earlier one can never be the choice (lowest index among equals) and would only tie with
    // it, so it leaves the scan.  (An earlier one behind another of the same hash stays unseen: its ties go to the
    // re-do like all others.)
    const int twin = (int)first_of[hash];
    bool again = twin < tid;
#pragma unroll
    for (int i = 0; i < C; ++i) again = again && cs[(twin >> 2) * QS + (twin & 3) * C + i] == own[i];
    norms[tid] = again ? -1.0e30f : (extreme ? 0.f : -0.5f * (n2 * f2));
    {
        const unsigned long long own_ones = __ballot(!again);
        if (lane == 0) kept[wave] = (unsigned)__popcll(own_ones);
    }
    __syncthreads();
    static_assert(kLloydWaves == 4, "the four counts");
    // (a single centroid wins every scan, whatever its size)
    const int distinct = __builtin_amdgcn_readfirstlane((int)(kept[0] + kept[1] + kept[2] + kept[3]));
    const bool group_direct = extreme && distinct > 1;

    // A operands: lane l holds row l % 32 of each block of 32 centroids; lanes below 32 the high
    // parts, the others the low parts (C = 2: both in the lower lanes).  D's registers: row
    // 8 (i / 4) + 4 (lane / 32) + i % 4.
    vec_t aop[kNBlk];
    // (the norms of every second block come from LDS where 128 registers for all of them are too many)
    constexpr bool HALF_LDS = MODE == kNext || (C == 8 && MODE != kPlain);
    float16_t nrm[kNBlk];
    auto load_norms = [&](int b, int row) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(&norms[row + b * 32 + 8 * q]);
            nrm[b][4 * q] = v.x; nrm[b][4 * q + 1] = v.y; nrm[b][4 * q + 2] = v.z; nrm[b][4 * q + 3] = v.w;
        }
    };
#pragma unroll
    for (int b = 0; b < kNBlk; ++b) {
        const int j = b * 32 + (lane & 31);
        float c[C];
#pragma unroll
        for (int i = 0; i < C; ++i) c[i] = group_direct ? 0.f : cs[(j >> 2) * QS + (j & 3) * C + i] * f1;
        _Float16 hi[C], lo[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            hi[i] = (_Float16)c[i];
            lo[i] = (_Float16)(c[i] - (float)hi[i]);
        }
        if constexpr (C == 2) {
            const _Float16 z = (_Float16)0.f;
            aop[b] = lane < 32 ? vec_t{hi[0], hi[1], lo[0], lo[1]} : vec_t{z, z, z, z};
        } else {
#pragma unroll
            for (int i = 0; i < C; ++i) aop[b][i] = lane < 32 ? hi[i] : lo[i];
        }
        if (!HALF_LDS || b % 2 == 0) load_norms(b, 4 * (lane >> 5));
    }

    auto cent_at = [&](int j, float (&c)[C]) {
        const float* p = &cs[(j >> 2) * QS + (j & 3) * C];
        if constexpr (C == 2) {
            const float2 v = *reinterpret_cast<const float2*>(p);
            c[0] = v.x; c[1] = v.y;
        } else {
#pragma unroll
            for (int i = 0; i < C / 4; ++i) {
                const float4 v = *reinterpret_cast<const float4*>(p + 4 * i);
                c[4 * i] = v.x; c[4 * i + 1] = v.y; c[4 * i + 2] = v.z; c[4 * i + 3] = v.w;
            }
        }
    };

    const int t_begin = split * tokens_per_split, t_end = min(t_begin + tokens_per_split, n);
    // (the unit of lengths in the state is that of the first iteration)
    const float to_state = MODE == kNext ? f0 / f1 : 1.f, c_longest = __builtin_amdgcn_sqrtf(c2s);
    // 64 tokens at a time: two sets of 32 as they are stored, xa of lanes % 32, xb of 32 + lanes % 32 (this lane's own
    // token: number i0, of cluster `old` so far, if `valid`).  request() is called once their words have been read.
    // What it finds is stored by put() ahead of the next request: a store behind it would be waited for with it.
    int put_at = -1;
    unsigned put_threshold = 0, put_cluster = 0;
    auto put = [&] {
        if (put_at < 0) return;
        const unsigned at = (unsigned)put_at;
        if constexpr (MODE != kPlain) threshold[at] = (uint16_t)put_threshold;
        if constexpr (MODE == kFirst) own_cluster[at] = (uint8_t)put_cluster;
        if (assign_now) assign_now[(size_t)g * n + at] = (uint16_t)put_cluster;
    };
    // ---- the clusters' sums: x 2^24 is an integer, hi 2^20 + lo with hi = floor(16 x).  A token joins cluster `to` and
    // (kNext) leaves cluster `from`.
    auto add_token = [&](const float (&x)[C], int i0, int from, int to) {
        unsigned long long* sj = &sums[to * SW];
        unsigned long long* so = &sums[from * SW];
        const auto move = [&](int i, unsigned long long v) {
            atomicAdd(sj + i, v);
            if constexpr (MODE == kNext) atomicAdd(so + i, 0ull - v);
        };
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if constexpr (W) {
                const float x16 = x[i] * 16.f, fl = __builtin_floorf(x16);
                const long long xhi = (long long)(int)fl, xlo = (long long)(int)((x16 - fl) * 1048576.f);
                const long long w = (long long)wq[i0];
                move(2 * i, (unsigned long long)(w * xhi));
                move(2 * i + 1, (unsigned long long)(w * xlo));
            } else {
                // 16 x and the rest in units of 2^-24 as the mantissas of 1.5 2^23 + (integer): exact, and
                // the constants of the bit patterns go back out with the count
                const float t = __builtin_fmaf(x[i], 16.f, kMagic);
                const float u = __builtin_fmaf(__builtin_fmaf(x[i], 16.f, kMagic - t), 1048576.f, kMagic);
                move(i, ((unsigned long long)__float_as_uint(t) << 20) + __float_as_uint(u));
            }
        }
        move(SW - 1, W ? (unsigned long long)wq[i0] : 1ull);
    };
    int n_changed = 0;                      // kNext: tokens of `changed` whose move is still to be made
    auto tokens = [&](unsigned (&xa)[C / 2], unsigned (&xb)[C / 2], int i0, int old, bool valid, auto&& request) {
        unsigned xw[C / 2], xs[2][C / 2];
#pragma unroll
        for (int i = 0; i < C / 2; ++i) {
            const unsigned wa = xa[i], wb = xb[i];
            xw[i] = lane < 32 ? wa : wb;
            xs[0][i] = __builtin_bit_cast(unsigned, __builtin_bit_cast(half2_t, wa) * m1 * m2);
            xs[1][i] = __builtin_bit_cast(unsigned, __builtin_bit_cast(half2_t, wb) * m1 * m2);
        }
        put();
        request();

        float x2 = 0.f;                                     // |x'|^2 of this lane's own token (infinite where the scaling overflowed)
#pragma unroll
        for (int i = 0; i < C / 2; ++i) {
            const unsigned sa = xs[0][i], sb = xs[1][i];
            const half2_t v = __builtin_bit_cast(half2_t, lane < 32 ? sa : sb);
            x2 = __builtin_amdgcn_fdot2(v, v, x2, false);
        }
        const bool direct = group_direct || !(x2 < 1.0e9f);
        const float slack = 0.01f * __builtin_amdgcn_sqrtf(c2s + x2);

        // ---- scan: the two largest maxima of eight, for tokens 32 h + lane % 32
        float hbest[2] = {LOWEST, LOWEST}, hsecond[2] = {LOWEST, LOWEST};
        vec_t bop[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (C == 8) {
                const half2_t p0 = __builtin_bit_cast(half2_t, xs[h][0]), p1 = __builtin_bit_cast(half2_t, xs[h][1]);
                const half2_t p2 = __builtin_bit_cast(half2_t, xs[h][2]), p3 = __builtin_bit_cast(half2_t, xs[h][3]);
                bop[h] = vec_t{p0.x, p0.y, p1.x, p1.y, p2.x, p2.y, p3.x, p3.y};
            } else if constexpr (C == 4) {
                const half2_t p0 = __builtin_bit_cast(half2_t, xs[h][0]), p1 = __builtin_bit_cast(half2_t, xs[h][1]);
                bop[h] = vec_t{p0.x, p0.y, p1.x, p1.y};
            } else {
                const half2_t p0 = __builtin_bit_cast(half2_t, xs[h][0]);
                bop[h] = vec_t{p0.x, p0.y, p0.x, p0.y};
            }
        }
        int norm_row = 4 * (lane >> 5);
        asm volatile("" : "+v"(norm_row));                   // (read again for every 64 tokens)
#pragma unroll
        for (int b = 0; b < kNBlk; ++b) {
            if (HALF_LDS && b % 2 == 0) load_norms(b + 1, norm_row);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float16_t d;
                if constexpr (C == 8) d = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop[b], bop[h], nrm[b], 0, 0, 0);
                else d = __builtin_amdgcn_mfma_f32_32x32x8f16(aop[b], bop[h], nrm[b], 0, 0, 0);
                float om[2];
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int r = 8 * o;
                    float m = fmaxf(fmaxf(d[r], d[r + 1]), d[r + 2]);
                    m = fmaxf(fmaxf(m, d[r + 3]), d[r + 4]);
                    m = fmaxf(fmaxf(m, d[r + 5]), d[r + 6]);
                    m = fmaxf(m, d[r + 7]);
                    om[o] = __uint_as_float((__float_as_uint(m) & 0xfffffff0u) | (unsigned)(2 * b + o));
                }
                // the runner-up of {best, second, k1, k2}, second <= best, is max(median(best, k1, k2), second)
                hsecond[h] = fmaxf(hsecond[h], __builtin_amdgcn_fmed3f(hbest[h], om[0], om[1]));
                hbest[h] = fmaxf(fmaxf(hbest[h], om[0]), om[1]);
            }
        }
        // each lane takes its own token: the scans of the two lanes that saw it, the rows of the lower and of the upper
        // lanes (a swap of the registers' halves: one instruction for both)
        auto halves = [](float a, float b, float& lower, float& upper) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
            lower = __uint_as_float(r[0]);
            upper = __uint_as_float(r[1]);
        };
        float gbest, obest, gsecond, osecond;
        halves(hbest[0], hbest[1], gbest, obest);
        halves(hsecond[0], hsecond[1], gsecond, osecond);
        const bool other = obest > gbest;
        const float best = fmaxf(gbest, obest);
        const float second = fmaxf(fmaxf(fminf(gbest, obest), gsecond), osecond);
        const unsigned bb = __float_as_uint(best);
        const int j0 = (int)(bb & 15u) * 16 + 4 * (other ? 1 : 0);
        const float gap = __uint_as_float(bb & 0xfffffff0u) - __uint_as_float(__float_as_uint(second) & 0xfffffff0u);
        // ---- the winner's eight centroids (j0 .. j0 + 3, j0 + 8 .. j0 + 11) in the direct form
        float x[C];
        widen_words<C>(xw, x);
        float dbest = 0.f, dsecond = 3.0e38f;
        int arg = j0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int j = j0 + (k & 3) + 8 * (k >> 2);
            float c[C];
            cent_at(j, c);
            const float d = dist2<C>(x, c);
            if (k == 0) {
                dbest = d;
            } else {
                if constexpr (MODE != kPlain) dsecond = __builtin_amdgcn_fmed3f(dbest, dsecond, d);
                arg = d < dbest ? j : arg;
                dbest = d < dbest ? d : dbest;
            }
        }

        // the bound: a centroid that could be as near as the winner, or that scored as high, has a norm of
        // at most reach
        const float xn = __builtin_amdgcn_sqrtf(x2);
        const float reach = 1.001f * (xn + __builtin_amdgcn_sqrtf(dbest * f2)) + slack;
        const float thr = 0x1p-20f * (11.1f * reach * (xn + 0.5f * reach) + 0.76f * x2);
        const bool unsure = valid && (direct || !(gap > thr));

        // ---- near ties: all centroids in the direct form, by the whole wavefront a token at a time, or
        // (many of them: duplicated points, dead channels) every lane its own token
        unsigned long long todo = __ballot(unsure);
        if (__popcll(todo) > 24) {
            // four centroids at a time, each with a nearest so far of its own: nothing waits for its neighbour
            float db[4];
            int fb[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                db[k] = 3.0e38f;
                fb[k] = 0;
            }
#pragma unroll (C == 8 ? 1 : 2)
            for (int f = 0; f < kK / 4; ++f) {
                float c[4][C], d[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) cent_at(4 * f + k, c[k]);
#pragma unroll
                for (int k = 0; k < 4; ++k) d[k] = 0.f;
#pragma unroll
                for (int i = 0; i < C; ++i)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float e = x[i] - c[k][i];
                        d[k] = __builtin_fmaf(e, e, d[k]);
                    }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    fb[k] = d[k] < db[k] ? f : fb[k];
                    db[k] = fminf(db[k], d[k]);
                }
            }
            int ag = 4 * fb[0];
            float dg = db[0];
#pragma unroll
            for (int k = 1; k < 4; ++k) {               // (equal distances: the lowest index)
                const int j = 4 * fb[k] + k;
                const bool nearer = db[k] < dg || (db[k] == dg && j < ag);
                ag = nearer ? j : ag;
                dg = nearer ? db[k] : dg;
            }
            arg = unsure ? ag : arg;
        } else {
            while (todo) {
                const int r = (int)__builtin_ctzll(todo);
                todo &= todo - 1;
                unsigned rw[C / 2];
#pragma unroll
                for (int i = 0; i < C / 2; ++i) rw[i] = (unsigned)__builtin_amdgcn_readlane((int)xw[i], r);
                float rx[C];
                widen_words<C>(rw, rx);
                unsigned dmin = ~0u, jmin = 0;
#pragma unroll
                for (int k = 0; k < kK / 64; ++k) {
                    const int j = lane + 64 * k;
                    float c[C];
                    cent_at(j, c);
                    const unsigned dj = __float_as_uint(dist2<C>(rx, c));
                    jmin = dj < dmin ? (unsigned)j : jmin;      // increasing j: the lowest index stays on ties
                    dmin = dj < dmin ? dj : dmin;
                }
                const unsigned wmin = wave_extreme_u32<false>(dmin);
                const unsigned long long holders = __ballot(dmin == wmin);
                unsigned code;
                if ((holders & (holders - 1)) == 0) code = (unsigned)__builtin_amdgcn_readlane((int)jmin, (int)__builtin_ctzll(holders));
                else code = wave_extreme_u32<false>(dmin == wmin ? jmin : ~0u);
                arg = lane == r ? (int)code : arg;
            }
        }
        arg &= kK - 1;

        // ---- the token's threshold ("Skipping"): how much farther the next nearest centroid is at least, less the
        // error of everything here, ahead of what the centroids have travelled so far
        if constexpr (MODE != kPlain) {
            const float err = 0x1p-20f * (11.1f * c_longest * (xn + 0.5f * c_longest) + 0.76f * x2);
            const float other2 = fminf(x2 - 2.f * (__uint_as_float(__float_as_uint(second) & 0xfffffff0u) + err), dsecond * f2 * (1.f - 0x1p-20f));
            const float to_other = __builtin_amdgcn_sqrtf(fmaxf(other2, 0.f)), to_own = __builtin_amdgcn_sqrtf(dbest * f2);
            const float ahead = (to_other - to_own) - 0x1p-18f * (to_other + to_own);
            const float moved = MODE == kNext ? need[arg] * (1.f - 0x1p-20f) : 0.f;
            const float t = unsure || distinct < kK || !(ahead > 0.f) ? 0.f : (ahead * to_state + moved) * (1.f - 0x1p-20f);
            put_threshold = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(t, t));     // (towards zero, at most 65504)
        }
        put_at = valid ? i0 : -1;
        put_cluster = (unsigned)arg;
        if constexpr (MODE == kNext) {
            const bool other_now = valid && arg != old;
            const unsigned long long mask = __ballot(other_now);
            if (other_now)
                changed[wave][n_changed + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u))] =
                    (unsigned)i0 | ((unsigned long long)((unsigned)old | ((unsigned)arg << 8)) << 32);
            n_changed += __popcll(mask);
        } else {
            if (valid) add_token(x, i0, 0, arg);
        }
    };
    // kNext: the moves of up to 64 changed tokens (one in twenty changes: together they cost what those of one would)
    auto make_moves = [&] {
        const int count = min(n_changed, 64);
        n_changed -= count;
        if (lane < count) {
            const unsigned long long e = changed[wave][n_changed + lane];
            const unsigned i0 = (unsigned)e, from = (unsigned)(e >> 32) & 255u, to = (unsigned)(e >> 40) & 255u;
            unsigned xw[C / 2];
            load_words<C>(reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(xg) + i0 * (2u * C)), xw);
            float x[C];
            widen_words<C>(xw, x);
            own_cluster[i0] = (uint8_t)to;
            add_token(x, (int)i0, (int)from, (int)to);
        }
    };

    if constexpr (MODE != kNext) {
        unsigned xa[C / 2], xb[C / 2];
        auto load_tile = [&](int at) {
            load_words<C>(xg + (size_t)min(at + (lane & 31), n - 1) * C, xa);
            load_words<C>(xg + (size_t)min(at + 32 + (lane & 31), n - 1) * C, xb);
        };
        int base = t_begin + wave * 64;
        load_tile(base);
#pragma unroll 1
        for (; base < t_end; base += kLloydWaves * 64)
            tokens(xa, xb, base + lane, 0, base + lane < t_end, [&] { load_tile(base + kLloydWaves * 64); });   // (clamped to the last token)
        put();
    } else {
        // Each wavefront has a quarter of the tokens to itself: it looks at the thresholds of 512 at a time, lists
        // the tokens that could have a new cluster, and takes 64 of the list at a time.  Thresholds and tokens are
        // requested one step ahead.
        const int share = ((t_end - t_begin + kLloydWaves - 1) / kLloydWaves + kScanTokens - 1) / kScanTokens * kScanTokens;
        int at = t_begin + wave * share;
        const int end = min(at + share, t_end);
        uint4 th;
        uint2 cl;
        auto load_thresholds = [&] {
            const size_t i = (size_t)min(at + kScanTokens * lane, state.n_pad - kScanTokens);
            th = *(const uint4*)(threshold + i);
            cl = *(const uint2*)(own_cluster + i);
        };
        load_thresholds();
        unsigned* todo_list = list[wave];
        unsigned xa[C / 2] = {}, xb[C / 2] = {}, ea = 0, eb = 0;
        int listed = 0, flying = 0;
#pragma unroll 1
        for (;;) {
            // (the tokens' words, requested long ago, are waited for ahead of the next thresholds' request)
            unsigned ya[C / 2], yb[C / 2];
#pragma unroll
            for (int i = 0; i < C / 2; ++i) {
                ya[i] = xa[i];
                yb[i] = xb[i];
                asm volatile("" : "+v"(ya[i]), "+v"(yb[i]));
            }
#pragma unroll 1
            while (listed < 64 && at < end) {
                const uint4 t4 = th;
                const uint2 c8 = cl;
                const int first = at + kScanTokens * lane;
                at += 64 * kScanTokens;
                load_thresholds();
#pragma unroll
                for (int k = 0; k < kScanTokens; ++k) {
                    const unsigned tw = k < 2 ? t4.x : k < 4 ? t4.y : k < 6 ? t4.z : t4.w, cw = k < 4 ? c8.x : c8.y;
                    const float t = (float)__builtin_bit_cast(half2_t, tw)[k & 1];
                    const unsigned c = (cw >> (8 * (k & 3))) & 255u;
                    const bool here = first + k < end, look = here && !(t > need[c]);
                    const unsigned long long mask = __ballot(look);
                    if (look) todo_list[listed + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u))] = (unsigned)(first + k) | (c << 24);
                    if (assign_now && here && !look) assign_now[(size_t)g * n + first + k] = (uint16_t)c;
                    listed += __popcll(mask);
                }
            }
            const int now = flying;
            const unsigned mine = lane < 32 ? ea : eb;
            auto request = [&] {
                flying = min(listed, 64);
                listed -= flying;
                if (flying) {                               // (lanes beyond the last one listed repeat it)
                    ea = todo_list[listed + min(lane & 31, flying - 1)];
                    eb = todo_list[listed + min(32 + (lane & 31), flying - 1)];
                    load_words<C>(reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(xg) + (ea & 0xffffffu) * (2u * C)), xa);
                    load_words<C>(reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(xg) + (eb & 0xffffffu) * (2u * C)), xb);
                }
            };
            if (now) tokens(ya, yb, (int)(mine & 0xffffffu), (int)(mine >> 24), lane < now, request);
            else request();
            if (n_changed >= 64) make_moves();
            if (!flying) break;
        }
        put();
        make_moves();
    }
    __syncthreads();
    if constexpr (MODE != kPlain) {
        // the group's sums so far and the changes of this launch; then each thread has a centroid
        if (!alone) {
            unsigned* flag = first_of;
            for (int i = tid; i < kK * SW; i += kLloydWaves * 64)
                if (sums[i] != 0ull) __hip_atomic_fetch_add(all_sums + i, sums[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // (all of them have been carried out)
            __syncthreads();
            if (tid == 0) {
                const bool last = __hip_atomic_fetch_add(state.arrived + g, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1u;
                if (last) __hip_atomic_store(state.arrived + g, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *flag = last;
            }
            __syncthreads();
            if (!*flag) return;
            for (int i = tid; i < kK * SW; i += kLloydWaves * 64) sums[i] = __hip_atomic_load(all_sums + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
        }
        const unsigned long long* sj = &sums[tid * SW];
        const long long wk = (long long)sj[SW - 1];
        float step2 = 0.f;
        bool moved = false;
        if (wk != 0) {                                      // a cluster without tokens keeps its centroid
#pragma unroll
            for (int i = 0; i < C; ++i) {
                float* at = &cs[(tid >> 2) * QS + (tid & 3) * C + i];
                const float v = W ? kmeans_mean((long long)sj[2 * i], (long long)sj[2 * i + 1], wk) : kmeans_mean(plain_sum(sj[i], sj[SW - 1]), wk);
                const float d = (v - *at) * (MODE == kNext ? f0 : f1);
                step2 = __builtin_fmaf(d, d, step2);
                moved = moved || __float_as_uint(v) != __float_as_uint(*at);
                *at = v;
            }
        }
        // (rounded up, so that no sum of steps comes out too short)
        const float step = moved ? fmaxf(__builtin_amdgcn_sqrtf(step2) * (1.f + 0x1p-16f), 0x1p-126f) : 0.f;
        if (step > 0.f) travelled = (travelled + step) * (1.f + 0x1p-22f);
        const unsigned wstep = wave_extreme_u32<true>(__float_as_uint(step));
        if (lane == 0) c2w[wave] = wstep;
        __syncthreads();
        float m = 0.f;
#pragma unroll
        for (int w = 0; w < kLloydWaves; ++w) m = fmaxf(m, __uint_as_float(c2w[w]));
        if (m > 0.f) longest = (longest + m) * (1.f + 0x1p-22f);
        const bool done = m == 0.f;                         // ("Skipping": every later iteration is this one again)
        if (last_iteration || done) {
#pragma unroll
            for (int i = 0; i < C; ++i) cent[(size_t)tid * C + i] = cs[(tid >> 2) * QS + (tid & 3) * C + i];
            travel[tid] = travelled;
            if (tid == 0) {
                travel[kK] = longest;
                travel[kK + 1] = MODE == kNext ? f0 : f1;
                travel[kK + 2] = done ? 1.f : 0.f;
            }
            if (alone) {                                    // (for the next launch)
                for (int i = tid; i < kK * SW; i += kLloydWaves * 64) all_sums[i] = sums[i];
            }
        }
        if (MODE == kNext && done && !last_iteration) {
            if (assign_all) write_assignment(0, n);
            break;
        }
    } else if (partials) {
        unsigned long long* dst = partials + ((size_t)g * gridDim.x + split) * (kK * SW);
        for (int i = tid; i < kK * SW; i += kLloydWaves * 64) dst[i] = sums[i];
    } else {
        for (int i = tid; i < kK * C; i += kLloydWaves * 64) {
            const int k = i / C, ch = i - k * C;
            const unsigned long long* sj = &sums[k * SW];
            const long long wk = (long long)sj[SW - 1];
            if (wk == 0) continue;                          // a cluster without tokens keeps its centroid
            cent[i] = W ? kmeans_mean((long long)sj[2 * ch], (long long)sj[2 * ch + 1], wk) : kmeans_mean(plain_sum(sj[ch], sj[SW - 1]), wk);
        }
    }
    if (MODE != kNext || last_iteration) break;
    __syncthreads();
    }
}

// the splits' sums -> the new centroids
template <int C, bool W>
__global__ __launch_bounds__(256) void kmeans_combine_kernel(const unsigned long long* partials, float* cent_all, int n_split)
{
    constexpr int SW = kSumWords<C, W>;
    const int g = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;       // i < 256 C
    const int k = i / C, ch = i - k * C;
    unsigned long long a = 0, b = 0, w = 0;
    for (int sp = 0; sp < n_split; ++sp) {
        const unsigned long long* sj = partials + (((size_t)g * n_split + sp) * kK + k) * SW;
        a += sj[W ? 2 * ch : ch];
        if constexpr (W) b += sj[2 * ch + 1];
        w += sj[SW - 1];
    }
    if ((long long)w == 0) return;
    cent_all[(size_t)g * kK * C + i] = W ? kmeans_mean((long long)a, (long long)b, (long long)w) : kmeans_mean(plain_sum(a, w), (long long)w);
}

__global__ __launch_bounds__(256) void kmeans_clear_words_kernel(unsigned* p, size_t words)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < words) p[i] = 0u;
}

template <int C, bool W>
cq_status launch_lloyd(const KMeansLloyd& a, hipStream_t st)
{
    // Groups are independent: two workgroups of four wavefronts fill a CU (256 registers each), so
    // G >= 512 groups need no split; fewer groups split their tokens as far as the sums of the
    // splits fit the scratch and a split keeps 16 tiles
    constexpr size_t kSums = sizeof(unsigned long long) * kK * kSumWords<C, W>;
    int wanted = a.groups >= 512 ? 1 : (512 + a.groups - 1) / a.groups;
    const int by_tokens = a.n / 1024, by_scratch = (int)(a.scratch_bytes / ((size_t)a.groups * kSums));
    wanted = wanted < by_tokens ? wanted : by_tokens;
    struct Split {
        int n, tokens;
        Split(int n_split, int tokens_all)
        {
            n_split = n_split < 1 ? 1 : n_split;
            tokens = ((tokens_all + n_split - 1) / n_split + 63) / 64 * 64;
            n = (tokens_all + tokens - 1) / tokens;
        }
    };

    // from iteration kPlainIterations on with state, where there are enough of them and the scratch holds it
    LloydState state = {};
    state.n_pad = (a.n + kScanTokens - 1) / kScanTokens * kScanTokens;
    const size_t G = (size_t)a.groups, cleared = G * (kSums + kTravelWords * sizeof(float) + sizeof(unsigned));
    const size_t threshold_at = (cleared + 15) / 16 * 16;
    const bool stateful = a.n_iter >= kStateIterations && a.n < (1 << 24) && threshold_at + G * state.n_pad * 3 <= a.scratch_bytes;
    const int plain = stateful ? kPlainIterations : a.n_iter;
    const dim3 block(kLloydWaves * 64);

    const Split ps(wanted < by_scratch ? wanted : by_scratch, a.n);
    unsigned long long* partials = ps.n > 1 ? static_cast<unsigned long long*>(a.scratch) : nullptr;
    for (int it = 0; it < plain; ++it) {
        hipLaunchKernelGGL((kmeans_lloyd_kernel<C, W, kPlain>), dim3(ps.n, a.groups), block, 0, st, a.xg, a.wq, a.cent,
                           it + 1 == a.n_iter ? a.assign : nullptr, partials, state, a.n, ps.tokens, 1);
        if (partials)
            hipLaunchKernelGGL((kmeans_combine_kernel<C, W>), dim3(C, a.groups), dim3(256), 0, st, partials, a.cent, ps.n);
    }
    if (stateful) {
        char* base = static_cast<char*>(a.scratch);
        state.sums = reinterpret_cast<unsigned long long*>(base);
        state.travel = reinterpret_cast<float*>(base + G * kSums);
        state.arrived = reinterpret_cast<unsigned*>(state.travel + G * kTravelWords);
        state.threshold = reinterpret_cast<uint16_t*>(base + threshold_at);
        state.own = reinterpret_cast<uint8_t*>(state.threshold + G * state.n_pad);
        hipLaunchKernelGGL(kmeans_clear_words_kernel, dim3((unsigned)((cleared / 4 + 255) / 256)), dim3(256), 0, st,
                           reinterpret_cast<unsigned*>(base), cleared / 4);
        const Split ss(wanted, a.n);
        const dim3 grid(ss.n, a.groups);
        unsigned long long* none = nullptr;
        hipLaunchKernelGGL((kmeans_lloyd_kernel<C, W, kFirst>), grid, block, 0, st, a.xg, a.wq, a.cent, static_cast<uint16_t*>(nullptr),
                           none, state, a.n, ss.tokens, 1);
        // A workgroup holds its CU (all registers of two wavefronts per SIMD) until its launch ends, and the caller sets the
        // number of iterations: the two bounds keep what other streams' work has to wait for to 15-40 ms, which is in
        // the range of the k-means++ launch ahead of it.  The bounds leave the usual 100 iterations over 32768 tokens whole: every cut
        // waits for the busiest group (32768 tokens, 512 groups, 89 iterations in two, three or six launches: 24.3 -> 24.8, 24.8 ->
        // 25.4, 25.9 -> 26.5 ms for the fit, weighted 28.7 -> 29.4, 29.3 -> 30.4, 31.0 -> 32.2).
        const int left = a.n_iter - plain - 1;
        const int by_length = a.n >= kLaunchTokens ? 1 : kLaunchTokens / a.n;
        const int most = ss.n > 1 ? 1 : by_length < kLaunchIterations ? by_length : kLaunchIterations;
        for (int it = 0; it < left; it += most) {
            const int now = left - it < most ? left - it : most;
            hipLaunchKernelGGL((kmeans_lloyd_kernel<C, W, kNext>), grid, block, 0, st, a.xg, a.wq, a.cent,
                               it + now == left ? a.assign : nullptr, none, state, a.n, ss.tokens, now);
        }
    }
    return hipGetLastError() == hipSuccess ? CQ_OK : CQ_ERR_HIP;
}

}  // namespace

cq_status launch_kmeans_lloyd(const KMeansLloyd& a, int c, hipStream_t stream)
{
    if (c == 8) return a.wq ? launch_lloyd<8, true>(a, stream) : launch_lloyd<8, false>(a, stream);
    if (c == 4) return a.wq ? launch_lloyd<4, true>(a, stream) : launch_lloyd<4, false>(a, stream);
    if (c == 2) return a.wq ? launch_lloyd<2, true>(a, stream) : launch_lloyd<2, false>(a, stream);
    return CQ_ERR_UNSUPPORTED;
}

}  // namespace cq
