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
// What bounds it: the vector ALU (535 instructions per 64 tokens and group: 208 in the scan, 150 in
// the winner's eight, the rest merge, bound, sums and re-dos; the direct search took 2 c + 3 per
// token and centroid).  The group's centroids sit in registers as matrix operands (32 registers)
// with the norms in accumulator layout (128): two wavefronts per SIMD and no LDS reads in the
// scan.  32768 tokens, 512 groups of 8 channels: 1.36 + 0.30 ms per iteration in two kernels ->
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

// One workgroup: tokens [split * tokens_per_split, ...) of one group.  One split per group: the new
// centroids are written at once; else the sums go to `partials` [group][split][256][kSumWords].
template <int C, bool W>
__global__ __launch_bounds__(kLloydWaves * 64, 2) void kmeans_lloyd_kernel(const uint16_t* __restrict__ xg_all,
                                                                        const uint32_t* __restrict__ wq_all,
                                                                        float* cent_all, uint16_t* __restrict__ assign_all,
                                                                        unsigned long long* __restrict__ partials, int n,
                                                                        int tokens_per_split)
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

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.y, split = blockIdx.x;
    const uint16_t* xg = xg_all + (size_t)g * n * C;
    const uint32_t* wq = W ? wq_all + (size_t)g * n : nullptr;
    float* cent = cent_all + (size_t)g * kK * C;

    // ---- the group's centroids: fp32 in LDS, scale, norms, matrix operands
    static_assert(kLloydWaves * 64 == kK, "one centroid per thread");
    float n2 = 0.f, own[C];
    unsigned hash = 0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        own[i] = cent[(size_t)tid * C + i];
        n2 = __builtin_fmaf(own[i], own[i], n2);
        cs[(tid >> 2) * QS + (tid & 3) * C + i] = own[i];
        hash = (hash ^ __float_as_uint(own[i] + 0.f)) * 0x9e3779b1u;        // (zeros of both signs are equal)
        hash ^= hash >> 15;
    }
    hash = (hash * 0x85ebca6bu) / (0xffffffffu / kHashSlots + 1u);
    for (int i = tid; i < kHashSlots; i += kLloydWaves * 64) first_of[i] = ~0u;
    const unsigned wmax = wave_extreme_u32<true>(__float_as_uint(n2));
    if (lane == 0) c2w[wave] = wmax;
    for (int i = tid; i < kK * SW; i += kLloydWaves * 64) sums[i] = 0ull;
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
    const bool group_direct = extreme && __builtin_amdgcn_readfirstlane((int)(kept[0] + kept[1] + kept[2] + kept[3])) > 1;

    // A operands: lane l holds row l % 32 of each block of 32 centroids; lanes below 32 the high
    // parts, the others the low parts (C = 2: both in the lower lanes).  D's registers: row
    // 8 (i / 4) + 4 (lane / 32) + i % 4.
    vec_t aop[kNBlk];
    float16_t nrm[kNBlk];
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
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(&norms[b * 32 + 8 * q + 4 * (lane >> 5)]);
            nrm[b][4 * q] = v.x; nrm[b][4 * q + 1] = v.y; nrm[b][4 * q + 2] = v.z; nrm[b][4 * q + 3] = v.w;
        }
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
    unsigned xa[C / 2], xb[C / 2];                          // tokens base + lane % 32 and base + 32 + lane % 32
    auto load_tile = [&](int at, unsigned (&lo)[C / 2], unsigned (&up)[C / 2]) {
        load_words<C>(xg + (size_t)min(at + (lane & 31), n - 1) * C, lo);
        load_words<C>(xg + (size_t)min(at + 32 + (lane & 31), n - 1) * C, up);
    };
    int base = t_begin + wave * 64;
    load_tile(base, xa, xb);
#pragma unroll 1
    for (; base < t_end; base += kLloydWaves * 64) {
        unsigned xw[C / 2], xs[2][C / 2];
#pragma unroll
        for (int i = 0; i < C / 2; ++i) {
            const unsigned wa = xa[i], wb = xb[i];
            xw[i] = lane < 32 ? wa : wb;
            xs[0][i] = __builtin_bit_cast(unsigned, __builtin_bit_cast(half2_t, wa) * m1 * m2);
            xs[1][i] = __builtin_bit_cast(unsigned, __builtin_bit_cast(half2_t, wb) * m1 * m2);
        }
        load_tile(base + kLloydWaves * 64, xa, xb);         // (clamped to the last token)

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
        float hbest[2], hsecond[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            vec_t bop;
            if constexpr (C == 8) {
                const half2_t p0 = __builtin_bit_cast(half2_t, xs[h][0]), p1 = __builtin_bit_cast(half2_t, xs[h][1]);
                const half2_t p2 = __builtin_bit_cast(half2_t, xs[h][2]), p3 = __builtin_bit_cast(half2_t, xs[h][3]);
                bop = vec_t{p0.x, p0.y, p1.x, p1.y, p2.x, p2.y, p3.x, p3.y};
            } else if constexpr (C == 4) {
                const half2_t p0 = __builtin_bit_cast(half2_t, xs[h][0]), p1 = __builtin_bit_cast(half2_t, xs[h][1]);
                bop = vec_t{p0.x, p0.y, p1.x, p1.y};
            } else {
                const half2_t p0 = __builtin_bit_cast(half2_t, xs[h][0]);
                bop = vec_t{p0.x, p0.y, p0.x, p0.y};
            }
            float best = LOWEST, second = LOWEST;
#pragma unroll
            for (int b = 0; b < kNBlk; ++b) {
                float16_t d;
                if constexpr (C == 8) d = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop[b], bop, nrm[b], 0, 0, 0);
                else d = __builtin_amdgcn_mfma_f32_32x32x8f16(aop[b], bop, nrm[b], 0, 0, 0);
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
                second = fmaxf(second, __builtin_amdgcn_fmed3f(best, om[0], om[1]));
                best = fmaxf(fmaxf(best, om[0]), om[1]);
            }
            hbest[h] = best;
            hsecond[h] = second;
        }
        // each lane takes its own token: its own scan of that half and the partner lane's (the other rows)
        const int hi = lane >> 5;
        const float gbest = hi ? hbest[1] : hbest[0], gsecond = hi ? hsecond[1] : hsecond[0];
        const float obest = __shfl_xor(hi ? hbest[0] : hbest[1], 32), osecond = __shfl_xor(hi ? hsecond[0] : hsecond[1], 32);
        const bool other = obest > gbest;
        const float best = fmaxf(gbest, obest);
        const float second = fmaxf(fmaxf(fminf(gbest, obest), gsecond), osecond);
        const unsigned bb = __float_as_uint(best);
        const int j0 = (int)(bb & 15u) * 16 + 4 * (other ? 1 - hi : hi);
        const float gap = __uint_as_float(bb & 0xfffffff0u) - __uint_as_float(__float_as_uint(second) & 0xfffffff0u);
        const bool valid = base + lane < t_end;

        // ---- the winner's eight centroids (j0 .. j0 + 3, j0 + 8 .. j0 + 11) in the direct form
        float x[C];
        widen_words<C>(xw, x);
        float dbest = 0.f;
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

        // ---- the cluster's sums: x 2^24 is an integer, hi 2^20 + lo with hi = floor(16 x)
        if (valid) {
            unsigned long long* sj = &sums[arg * SW];
            const int i0 = base + lane;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                if constexpr (W) {
                    const float x16 = x[i] * 16.f, fl = __builtin_floorf(x16);
                    const long long xhi = (long long)(int)fl, xlo = (long long)(int)((x16 - fl) * 1048576.f);
                    const long long w = (long long)wq[i0];
                    atomicAdd(sj + 2 * i, (unsigned long long)(w * xhi));
                    atomicAdd(sj + 2 * i + 1, (unsigned long long)(w * xlo));
                } else {
                    // 16 x and the rest in units of 2^-24 as the mantissas of 1.5 2^23 + (integer): exact, and
                    // the constants of the bit patterns go back out with the count
                    const float t = __builtin_fmaf(x[i], 16.f, kMagic);
                    const float u = __builtin_fmaf(__builtin_fmaf(x[i], 16.f, kMagic - t), 1048576.f, kMagic);
                    atomicAdd(sj + i, ((unsigned long long)__float_as_uint(t) << 20) + __float_as_uint(u));
                }
            }
            atomicAdd(sj + SW - 1, W ? (unsigned long long)wq[i0] : 1ull);
            if (assign_all) assign_all[(size_t)g * n + i0] = (uint16_t)arg;
        }
    }
    __syncthreads();
    if (partials) {
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

template <int C, bool W>
cq_status launch_lloyd(const KMeansLloyd& a, hipStream_t st)
{
    // Groups are independent: two workgroups of four wavefronts fill a CU (256 registers each), so
    // G >= 512 groups need no split; fewer groups split their tokens as far as the sums of the
    // splits fit the scratch and a split keeps 16 tiles
    constexpr size_t kSums = sizeof(unsigned long long) * kK * kSumWords<C, W>;
    int n_split = a.groups >= 512 ? 1 : (512 + a.groups - 1) / a.groups;
    const int by_tokens = a.n / 1024, by_scratch = (int)(a.scratch_bytes / ((size_t)a.groups * kSums));
    n_split = n_split < by_tokens ? n_split : by_tokens;
    n_split = n_split < by_scratch ? n_split : by_scratch;
    n_split = n_split < 1 ? 1 : n_split;
    const int tps = ((a.n + n_split - 1) / n_split + 63) / 64 * 64;
    n_split = (a.n + tps - 1) / tps;
    unsigned long long* partials = n_split > 1 ? static_cast<unsigned long long*>(a.scratch) : nullptr;
    for (int it = 0; it < a.n_iter; ++it) {
        uint16_t* assign = it + 1 == a.n_iter ? a.assign : nullptr;
        hipLaunchKernelGGL((kmeans_lloyd_kernel<C, W>), dim3(n_split, a.groups), dim3(kLloydWaves * 64), 0, st, a.xg, a.wq, a.cent,
                           assign, partials, a.n, tps);
        if (partials)
            hipLaunchKernelGGL((kmeans_combine_kernel<C, W>), dim3(C, a.groups), dim3(256), 0, st, partials, a.cent, n_split);
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
