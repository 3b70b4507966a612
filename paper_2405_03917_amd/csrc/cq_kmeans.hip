// Centroid learning of CQ (Section 3.2 of the paper, "Centroid Learning"): one independent
// k-means run per channel group (Eq. 5), k-means++ initialisation and a fixed number of Lloyd
// iterations (Section 4.3), optionally weighted per (token, group) as in the Fisher-guided
// objective of Eq. 6 (weighted k-means), for gfx950.
//
// Every decision of the iteration is taken in arithmetic that does not depend on the order in
// which tokens are processed, so that the result is reproducible bit for bit:
//   distance     sum_i (x_i - c_i)^2 in fp32: rounded difference, one fused multiply-add per
//                channel in channel order; x is fp16 widened, c an fp32 centroid
//   assignment   smallest distance, lowest index among equals
//   weights      integers wq = floor(w * 2^kw), the largest weight of a group in [2^21, 2^22)
//                (no weights, or all zero: wq = 1)
//   update       exact integer sums of wq * (x * 2^24), held as S_hi * 2^20 + S_lo in two 64-bit
//                integers, and of wq; centroid = fp32((fp64(S_hi) * 2^20 + fp64(S_lo)) / fp64(W)
//                * 2^-24); a cluster without tokens keeps its centroid
//   k-means++    first centre with probability wq / sum wq, the others with probability
//                proportional to wq * dmin (dmin: fp32 distance to the nearest centre so far),
//                sampled on integers: q = floor(fp64(wq) * fp64(dmin) * 2^kq), kq = 62 -
//                ceil(log2 n) - (exponent of the largest product + 1); r = floor(rnd * sum q /
//                2^64) with the caller's 64-bit random word of the pick; chosen = first token
//                whose inclusive prefix sum of q exceeds r; all products zero: floor(rnd * n / 2^64)
//
// Kernels: prepare (group-major copy of the tokens, integer weights), k-means++ (one workgroup
// per group, K sequential picks), and per Lloyd iteration the matrix-core kernel of
// cq_kmeans_mfma.hip where a group has 256 centroids of two or more channels; else an assignment
// kernel (plain fp32 VALU search against the group's centroids in LDS) and an update kernel
// (integer LDS atomics, then the new centroids).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "cq_kmeans_common.hpp"
#include "cq_kmeans_mfma.hpp"

namespace cq {
namespace {

constexpr int kPPThreads = 1024;     // k-means++ workgroup
constexpr int kAssignThreads = 256;
constexpr int kAssignPoints = 2;     // tokens per thread of the assignment kernel
constexpr int kUpdateClusters = 256; // clusters per update workgroup

// ------------------------------------------------------------------------------------------
// prepare
// ------------------------------------------------------------------------------------------
__global__ void kmeans_clear_kernel(unsigned* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// largest weight of every group (weights are non-negative: their bits order like their values)
__global__ void kmeans_wmax_kernel(const float* w, int n, int G, unsigned* wmax_bits)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= G) return;
    unsigned m = 0;
    for (int i = blockIdx.y; i < n; i += gridDim.y) {
        const unsigned b = __float_as_uint(w[(size_t)i * G + g]);
        m = b > m ? b : m;
    }
    atomicMax(wmax_bits + g, m);
}

// xg[g][i][:] = x[i][g c ..], wq[g][i] = integer weight.  A workgroup moves a tile of 32 tokens x
// 64 groups through LDS so that both sides are read and written in contiguous runs.
constexpr int kPrepTokens = 32, kPrepGroups = 64;

template <int C>
__global__ __launch_bounds__(256) void kmeans_prepare_kernel(const uint16_t* x, int64_t x_stride, const float* w,
                                                             const unsigned* wmax_bits, int n, int G, uint16_t* xg,
                                                             uint32_t* wq)
{
    using unit_t = std::conditional_t<C == 8, uint4, std::conditional_t<C == 4, uint2, std::conditional_t<C == 2, unsigned, uint16_t>>>;
    __shared__ unit_t tile[kPrepTokens][kPrepGroups + 1];
    __shared__ uint32_t wt[kPrepTokens][kPrepGroups + 1];
    const int i0 = blockIdx.x * kPrepTokens, g0 = blockIdx.y * kPrepGroups;
    {
        const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;     // tx: group, ty: token row
        for (int r = ty; r < kPrepTokens; r += 4) {
            const int i = i0 + r, g = g0 + tx;
            if (i < n && g < G) {
                tile[r][tx] = *reinterpret_cast<const unit_t*>(x + (size_t)i * x_stride + (size_t)g * C);
                uint32_t q = 1u;
                const unsigned mb = w ? wmax_bits[g] : 0u;
                if (mb != 0u) {
                    // kw = 21 - floor(log2(wmax)); w * 2^kw is exact in fp64, the conversion truncates
                    const int kw = 21 - ilogbf(__uint_as_float(mb));
                    q = (uint32_t)ldexp((double)w[(size_t)i * G + g], kw);
                }
                wt[r][tx] = q;
            }
        }
    }
    __syncthreads();
    {
        const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;     // tx: token, ty: group row
        for (int r = ty; r < kPrepGroups; r += 8) {
            const int g = g0 + r, i = i0 + tx;
            if (i < n && g < G) {
                *reinterpret_cast<unit_t*>(xg + ((size_t)g * n + i) * C) = tile[tx][r];
                wq[(size_t)g * n + i] = wt[tx][r];
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// k-means++
// ------------------------------------------------------------------------------------------
// 64-bit sums over a wavefront with data-parallel-primitive moves (all 64 lanes active): a few
// cycles per step where a shuffle through LDS costs more than a hundred.
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v)      // lanes without a source read 0
{
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, 0xf, 0xf, true);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long readlane_u64(unsigned long long v, int l)
{
    return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), l) << 32) |
           (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, l);
}
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
    v += dpp_u64<0xB1>(v);       // quad_perm [1,0,3,2]
    v += dpp_u64<0x4E>(v);       // quad_perm [2,3,0,1]
    v += dpp_u64<0x141>(v);      // row_half_mirror
    v += dpp_u64<0x140>(v);      // row_mirror
    return (readlane_u64(v, 0) + readlane_u64(v, 16)) + (readlane_u64(v, 32) + readlane_u64(v, 48));
}
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v)
{
    auto up = [](unsigned long long a, unsigned long long b) { return b > a ? b : a; };
    v = up(v, dpp_u64<0xB1>(v));
    v = up(v, dpp_u64<0x4E>(v));
    v = up(v, dpp_u64<0x141>(v));
    v = up(v, dpp_u64<0x140>(v));
    return up(up(readlane_u64(v, 0), readlane_u64(v, 16)), up(readlane_u64(v, 32), readlane_u64(v, 48)));
}
__device__ __forceinline__ unsigned long long wave_incl_scan_u64(unsigned long long v, int lane)
{
    v += dpp_u64<0x111>(v);      // row_shr 1, 2, 4, 8: sums within the row of 16 lanes
    v += dpp_u64<0x112>(v);
    v += dpp_u64<0x114>(v);
    v += dpp_u64<0x118>(v);
    const unsigned long long r0 = readlane_u64(v, 15), r1 = r0 + readlane_u64(v, 31), r2 = r1 + readlane_u64(v, 47);
    const int row = lane >> 4;
    return v + (row == 0 ? 0ull : row == 1 ? r0 : row == 2 ? r1 : r2);
}

// One workgroup per group.  Wavefront w owns the contiguous tokens [w W, (w + 1) W), W a multiple
// of 64; in round p its lane l handles token w W + 64 p + l, so every load is one contiguous run
// and (wavefront, round, lane) order is token order.  A pick: the wavefronts' totals locate the
// wavefront that holds the r-th unit of mass, that wavefront walks its rounds to the round, and
// a scan over its lanes finds the token.
template <int C>
__global__ __launch_bounds__(kPPThreads) void kmeanspp_kernel(const uint16_t* __restrict__ xg_all,
                                                              const uint32_t* __restrict__ wq_all,
                                                              float* __restrict__ dmin_all,
                                                              const uint64_t* __restrict__ rnd_all,
                                                              int32_t* __restrict__ picks_all, float* __restrict__ cent_all,
                                                              int n, int K, int log2n)
{
    constexpr int NWAVE = kPPThreads / 64;
    __shared__ unsigned long long wave_tot[NWAVE];
    __shared__ unsigned long long pmax_bits;
    __shared__ int pick_sh;

    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint16_t* xg = xg_all + (size_t)g * n * C;
    const uint32_t* wq = wq_all + (size_t)g * n;
    float* dmin = dmin_all + (size_t)g * n;
    const uint64_t* rnd = rnd_all + (size_t)g * K;
    int32_t* picks = picks_all ? picks_all + (size_t)g * K : nullptr;
    float* cent = cent_all + (size_t)g * K * C;

    const int rounds = (n + kPPThreads - 1) / kPPThreads;    // rounds of 64 tokens per wavefront
    const int t0 = wave * rounds * 64;                       // this wavefront's first token

    // q of this lane's token in round p: the integer weight (kq < -9000: first pick) or
    // floor(wq * dmin * 2^kq)
    auto mass = [&](int p, int kq) -> unsigned long long {
        const int i = t0 + p * 64 + lane;
        if (i >= n) return 0ull;
        if (kq < -9000) return wq[i];
        return (unsigned long long)ldexp((double)wq[i] * (double)dmin[i], kq);
    };
    // draws the token that holds unit r of the total mass (all threads call; sets pick_sh)
    auto draw = [&](uint64_t word, int kq) {
        unsigned long long local = 0;
        for (int p = 0; p < rounds; ++p) local += mass(p, kq);
        const unsigned long long wtot = wave_sum_u64(local);
        if (lane == 0) wave_tot[wave] = wtot;
        __syncthreads();
        unsigned long long off = 0, total = 0;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) {
            const unsigned long long t = wave_tot[w];
            off += w < wave ? t : 0ull;
            total += t;
        }
        const unsigned long long r = __umul64hi(word, total);
        if (r >= off && r < off + wtot) {                    // wavefront-uniform: exactly one wavefront
            unsigned long long run = off;
            for (int p = 0; p < rounds; ++p) {
                const unsigned long long q = mass(p, kq);
                const unsigned long long rsum = wave_sum_u64(q);
                if (run + rsum > r) {
                    const unsigned long long incl = run + wave_incl_scan_u64(q, lane);
                    const unsigned long long hit = __ballot(incl > r);
                    if (lane == 0) pick_sh = t0 + p * 64 + __builtin_ctzll(hit);
                    break;
                }
                run += rsum;
            }
        }
        __syncthreads();
    };

    draw(rnd[0], -10000);                                    // first centre: proportional to the integer weights
    for (int j = 0;; ++j) {
        const int pick = pick_sh;
        __syncthreads();                                     // everyone has read pick_sh
        if (tid == 0) {
            if (picks) picks[j] = pick;
            pmax_bits = 0ull;
        }
        float cj[C];
        widen<C>(xg + (size_t)pick * C, cj);
        if (tid < C) cent[(size_t)j * C + tid] = cj[tid];
        if (j + 1 == K) break;

        // distance to the nearest centre so far; largest weighted distance (non-negative doubles
        // order like their bits)
        double pmax = 0.0;
#pragma unroll 4
        for (int p = 0; p < rounds; ++p) {
            const int i = t0 + p * 64 + lane;
            if (i < n) {
                float xi[C];
                widen<C>(xg + (size_t)i * C, xi);
                const float d = dist2<C>(xi, cj);
                const float dm = (j == 0 || d < dmin[i]) ? d : dmin[i];
                dmin[i] = dm;
                const double pr = (double)wq[i] * (double)dm;
                pmax = pr > pmax ? pr : pmax;
            }
        }
        unsigned long long pb = (unsigned long long)__double_as_longlong(pmax);
        pb = wave_max_u64(pb);
        __syncthreads();                                     // pmax_bits was cleared; dmin is written
        if (lane == 0) atomicMax(&pmax_bits, pb);
        __syncthreads();
        const unsigned long long pm = pmax_bits;
        if (pm == 0ull) {                                    // every token sits on a centre already
            if (tid == 0) pick_sh = (int)__umul64hi(rnd[j + 1], (unsigned long long)n);
            __syncthreads();
            continue;
        }
        const int kq = 62 - log2n - ((int)((pm >> 52) & 0x7ffull) - 1023 + 1);
        draw(rnd[j + 1], kq);
    }
}

// The same picks with the distances to the nearest centre in registers, for up to 32 rounds of 1024
// tokens: the form above walks three arrays in L2 and HBM per pick, and the walk
// of one wavefront to the chosen token is a chain of 32 reductions.  Here wavefront w still owns
// the contiguous tokens [w W, (w + 1) W); a token's slice x is read again for every pick -- from
// registers (the first kRegRounds rounds), from LDS (the next kLdsRounds) or from memory (the
// rest, requested before the pick is known) -- and a pick is three barriers: the largest
// weighted distance, the wavefronts' masses, the token.  The owner of the r-th unit of mass keeps
// its mass in up to four sums, so the search is 4 + R / 4 independent reductions and one scan.
// Weights sit in registers too, 32 rounds of them in LDS (as 32 more registers they spilled 50 to 61).
// 32768 tokens, 512 groups of 8 channels, 256 picks: 30.6 ms -> 6.7 ms, weighted 30.7 -> 9.0 (and see draw() and visit()
// for the vector instructions, which bound it: 6.7-7.0 -> 5.4-6.4, at 12000 tokens 3.6 -> 2.9); 1500 tokens, 256
// groups of 4: 1.05 -> 0.71 ms; 100 tokens 0.54 -> 0.56 (two barriers' worth of other wavefronts' numbers), so that
// up to 128 go to the general kernel (run_kmeanspp).
// Slices of 4 (of 2: 8) weighted tokens per lane in registers instead of 2 (4), 32 rounds: 8 channels 11.0 -> 9.0 ms
// at 512 groups, 4 channels 3.7 -> 4.6 ms at 256 groups (spills).
// Unweighted slices of 4 channels: 14 per lane instead of 8, so that all 32 rounds are held, 8.36 -> 8.24 ms at 1024 groups; of 8
// channels 5 instead of 4: 5.8 -> 6.05 at 512 groups.
constexpr int kPPRounds = 32;
constexpr int min_of(int a, int b) { return a < b ? a : b; }
template <bool W, int R>
constexpr bool kPPWeightsInLds = W && R == kPPRounds;
template <int C, bool W, int R>
constexpr int kPPRegRounds = min_of(R, (W && !(C == 8 && kPPWeightsInLds<W, R>) ? 8 : !W && C == 4 ? 28 : 16) / (C / 2));
template <int C, bool W, int R>
constexpr int kPPLdsRounds = min_of(R - kPPRegRounds<C, W, R>, (kPPWeightsInLds<W, R> ? 15 : 72) / C);     // at most 144 KB, or 30 next to the weights

// floor(m 2^sh) of an integer below 2^46 (the result fits 62 bits)
__device__ __forceinline__ unsigned long long shift_floor(unsigned long long m, int sh)
{
    const int l = sh > 0 ? sh : 0, r = sh < 0 ? (-sh < 63 ? -sh : 63) : 0;
    return (m << l) >> r;
}

template <int C, bool W, int R>
__global__ __launch_bounds__(kPPThreads, 4) void kmeanspp_resident_kernel(const uint16_t* __restrict__ xg_all,
                                                                      const uint32_t* __restrict__ wq_all,
                                                                      const uint64_t* __restrict__ rnd_all,
                                                                      int32_t* __restrict__ picks_all,
                                                                      float* __restrict__ cent_all, int n, int K, int log2n)
{
    constexpr int NWAVE = kPPThreads / 64;
    constexpr int XW = C / 2;                                // words of a token's slice
    constexpr int kRegRounds = kPPRegRounds<C, W, R>;
    constexpr int kLdsRounds = kPPLdsRounds<C, W, R>;
    constexpr int kHeld = kRegRounds + kLdsRounds;
    constexpr bool WL = kPPWeightsInLds<W, R>, WR = W && !WL;
    constexpr int kSegs = min_of(R, 4);
    constexpr int kBatch = 4;                                // rounds requested together
    extern __shared__ __attribute__((aligned(16))) unsigned xl[];       // [kLdsRounds][1024][XW], the weights [R][1024] if here, the exchange slots
    unsigned* const wl = xl + (size_t)kLdsRounds * kPPThreads * XW;
    unsigned long long* const wave_tot = reinterpret_cast<unsigned long long*>(wl + (WL ? R * kPPThreads : 0));
    unsigned long long* const wave_max = wave_tot + NWAVE;
    int& pick_sh = *reinterpret_cast<int*>(wave_max + NWAVE);

    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint16_t* xg = xg_all + (size_t)g * n * C;
    const uint64_t* rnd = rnd_all + (size_t)g * K;
    int32_t* picks = picks_all ? picks_all + (size_t)g * K : nullptr;
    float* cent = cent_all + (size_t)g * K * C;
    const int rounds = (n + kPPThreads - 1) / kPPThreads;    // at most R
    const int t0 = wave * rounds * 64;

    int first = t0 + lane;                                   // this lane's token of round 0
    auto load_words = [&](int p, unsigned (&w)[XW]) {        // token of round p (clamped to the last)
        const unsigned* src = reinterpret_cast<const unsigned*>(reinterpret_cast<const char*>(xg) +
                                                                (unsigned)min(first + p * 64, n - 1) * (unsigned)(2 * C));
        if constexpr (XW == 4) {
            const uint4 v = *reinterpret_cast<const uint4*>(src);
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        } else if constexpr (XW == 2) {
            const uint2 v = *reinterpret_cast<const uint2*>(src);
            w[0] = v.x; w[1] = v.y;
        } else {
            w[0] = src[0];
        }
    };

    unsigned dmin[R];                                        // bits of the fp32 distance (they order like it); 0 where
                                                             // there is no token: no mass, never the largest
    unsigned wr[WR ? R : 1];
    auto weight = [&](int p) -> unsigned { return WL ? wl[p * kPPThreads + tid] : (W ? wr[WR ? p : 0] : 1u); };
    unsigned xr[kRegRounds][XW];
#pragma unroll
    for (int p = 0; p < R; ++p) {
        const int i = t0 + p * 64 + lane;
        const bool there = p < rounds && i < n;
        dmin[p] = there ? 0x7f800000u : 0u;
        if constexpr (W) {
            const unsigned w = there ? wq_all[(size_t)g * n + i] : 0u;
            if constexpr (WL) wl[p * kPPThreads + tid] = w;
            else wr[p] = w;
        }
        if (p < kRegRounds) {
            load_words(p, xr[p < kRegRounds ? p : 0]);
        } else if (p < kHeld) {
            unsigned w[XW];
            load_words(p, w);
#pragma unroll
            for (int i2 = 0; i2 < XW; ++i2) xl[((p - kRegRounds) * kPPThreads + tid) * XW + i2] = w[i2];
        }
    }

    // mass of this lane's token of round p: the weight itself (first pick) or floor(weight dmin 2^kq)
    auto mass_of = [&](unsigned b, unsigned w, int kq) -> unsigned long long {
        if (W && kq < -9000) return w;
        const unsigned ex = b >> 23, fr = b & 0x7fffffu;
        const unsigned m = ex ? fr | 0x800000u : fr;
        const int sh = (int)(ex ? ex : 1u) - 150 + kq;
        return shift_floor(W ? (unsigned long long)w * m : (unsigned long long)m, sh);
    };
    auto draw = [&](uint64_t word, int kq) {
        unsigned long long seg[kSegs];
        // A mass without weight is v = dmin 2^kq < 2^(62 - log2n) rounded down: 2^(63 - log2n) + v rounds v to units of
        // 2^(40 - log2n) (hi: the sum's mantissa), the rest lo is exact, at most half a unit and signed; both sums of a
        // segment fit 32 bits from 1025 tokens on.  Distances that are not finite or whose 2^kq is not an fp32 number
        // go the general way.  Eight instructions per token instead of about 20 (with v_fma_mix_f32 below, one iteration
        // after the picks: 12000 tokens of 512 groups of 8 channels 3.90 -> 3.17 ms, 16385 6.88 -> 5.45, of 2 channels, 2048 groups 18.0 -> 13.3).
        const bool split = !W && R > 1 && kq >= -126 && kq <= 100;
        if (split) {
            const float unit = __uint_as_float((unsigned)(127 + kq) << 23);
            const unsigned big_bits = (unsigned)(127 + 63 - log2n) << 23;
            const float big = __uint_as_float(big_bits);
#pragma unroll
            for (int s = 0; s < kSegs; ++s) {
                unsigned hi = 0;
                int lo = 0;
#pragma unroll
                for (int k = 0; k < R / kSegs; ++k) {
                    const float v = __uint_as_float(dmin[s * (R / kSegs) + k]) * unit, t = v + big;
                    hi += __float_as_uint(t) - big_bits;
                    lo += (int)__builtin_floorf(v - (t - big));
                }
                seg[s] = ((unsigned long long)hi << (40 - log2n)) + (unsigned long long)(long long)lo;
            }
        } else {
#pragma unroll
            for (int s = 0; s < kSegs; ++s) {
                seg[s] = 0;
#pragma unroll
                for (int k = 0; k < R / kSegs; ++k) {
                    const int p = s * (R / kSegs) + k;
                    seg[s] += mass_of(dmin[p], weight(p), kq);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        unsigned long long mass = seg[0];
#pragma unroll
        for (int s = 1; s < kSegs; ++s) mass += seg[s];
        const unsigned long long wtot = wave_sum_u64(mass);
        if (lane == 0) wave_tot[wave] = wtot;
        __syncthreads();
        unsigned long long off = 0, total = 0;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) {
            const unsigned long long t = wave_tot[w];
            off += w < wave ? t : 0ull;
            total += t;
        }
        const unsigned long long r = __umul64hi(word, total);
        if (r >= off && r < off + wtot) {                    // exactly one wavefront
            unsigned long long run = off;
            int s_hit = 0;
            {
                unsigned long long st[kSegs];
#pragma unroll
                for (int s = 0; s < kSegs; ++s) st[s] = wave_sum_u64(seg[s]);
#pragma unroll
                for (int s = 0; s + 1 < kSegs; ++s)
                    if (s_hit == s && run + st[s] <= r) { run += st[s]; s_hit = s + 1; }
            }
            s_hit = __builtin_amdgcn_readfirstlane(s_hit);
            constexpr int RS = R / kSegs;
            unsigned sd[RS], sw[RS];
#pragma unroll
            for (int s = 0; s < kSegs; ++s)
                if (s_hit == s) {
#pragma unroll
                    for (int k = 0; k < RS; ++k) {
                        sd[k] = dmin[s * RS + k];
                        if constexpr (!WL) sw[k] = weight(s * RS + k);
                    }
                }
            if constexpr (WL) {
#pragma unroll
                for (int k = 0; k < RS; ++k) sw[k] = weight(s_hit * RS + k);
            }
            unsigned long long q[RS], qt[RS];
#pragma unroll
            for (int k = 0; k < RS; ++k) {
                q[k] = mass_of(sd[k], sw[k], kq);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int k = 0; k < RS; ++k) qt[k] = wave_sum_u64(q[k]);
            int k_hit = 0;
            unsigned long long qh = q[0];
#pragma unroll
            for (int k = 0; k + 1 < RS; ++k)
                if (k_hit == k && run + qt[k] <= r) { run += qt[k]; k_hit = k + 1; qh = q[k + 1]; }
            const unsigned long long incl = run + wave_incl_scan_u64(qh, lane);
            const unsigned long long hit = __ballot(incl > r);
            if (lane == 0) pick_sh = t0 + (s_hit * RS + k_hit) * 64 + __builtin_ctzll(hit);
        }
        __syncthreads();
    };

    if constexpr (W) {
        draw(rnd[0], -10000);                                // first centre: proportional to the integer weights
    } else {
        if (tid == 0) pick_sh = (int)__umul64hi(rnd[0], (unsigned long long)n);
        __syncthreads();
    }
    for (int j = 0;; ++j) {
        // (opaque per pick: left alone, the compiler widens the held slices and forms the addresses of
        // all rounds once, ahead of this loop, and spills them)
        asm volatile("" : "+v"(first));
#pragma unroll
        for (int p = 0; p < kRegRounds; ++p)
#pragma unroll
            for (int i2 = 0; i2 < XW; ++i2) asm volatile("" : "+v"(xr[p][i2]));
        // the first tokens from memory are on their way before the pick's own centre is
        unsigned xb[kBatch][XW];
        if constexpr (kHeld < R) {
#pragma unroll
            for (int k = 0; k < kBatch; ++k) load_words(kHeld + k, xb[k]);
        }
        const int pick = pick_sh;
        float cj[C];
        widen<C>(xg + (size_t)pick * C, cj);
        if (tid == 0 && picks) picks[j] = pick;
        if (tid == 0) {
#pragma unroll
            for (int i = 0; i < C; ++i) cent[(size_t)j * C + i] = cj[i];
        }
        if (j + 1 == K) break;

        double pmax = 0.0;
        unsigned fmx = 0;
        auto visit = [&](const unsigned (&w)[XW], unsigned& dm, unsigned wgt) {
            if constexpr (W) {
                float xi[C];
#pragma unroll
                for (int i = 0; i < XW; ++i) {
                    const half2_t h = __builtin_bit_cast(half2_t, w[i]);
                    xi[2 * i] = (float)h.x;
                    xi[2 * i + 1] = (float)h.y;
                }
                dm = min(__float_as_uint(dist2<C>(xi, cj)), dm);
            } else {
                // x - c in one v_fma_mix_f32: conversion and subtraction, the same single rounding (with weights 512 groups
                // of 8 channels were slower by it, 9.0 -> 10.6 ms at 16385 tokens, others 1-8 % faster)
                float acc = 0.f;
#pragma unroll
                for (int i = 0; i < XW; ++i) {
                    float d0, d1;
                    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(d0) : "v"(w[i]), "v"(cj[2 * i]));
                    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d1) : "v"(w[i]), "v"(cj[2 * i + 1]));
                    acc = __builtin_fmaf(d0, d0, acc);
                    acc = __builtin_fmaf(d1, d1, acc);
                }
                dm = min(__float_as_uint(acc), dm);
            }
            if constexpr (W) {
                const double pr = (double)wgt * (double)__uint_as_float(dm);
                pmax = pr > pmax ? pr : pmax;
            } else {
                fmx = max(fmx, dm);
            }
        };
#pragma unroll
        for (int p = 0; p < kHeld; ++p) {
            unsigned w[XW];
#pragma unroll
            for (int i2 = 0; i2 < XW; ++i2)
                w[i2] = p < kRegRounds ? xr[p < kRegRounds ? p : 0][i2] : xl[((p - kRegRounds) * kPPThreads + tid) * XW + i2];
            visit(w, dmin[p], weight(p));
            __builtin_amdgcn_sched_barrier(0);               // (one round's widened channels live at a time)
        }
#pragma unroll
        for (int p = kHeld; p < R; p += kBatch) {
            unsigned xn[kBatch][XW];
            if (p + kBatch < R) {
#pragma unroll
                for (int k = 0; k < kBatch; ++k) load_words(p + kBatch + k, xn[k]);
            }
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                if (p + k < R) visit(xb[k], dmin[p + k < R ? p + k : 0], weight(p + k < R ? p + k : 0));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (p + kBatch < R) {
#pragma unroll
                for (int k = 0; k < kBatch; ++k)
#pragma unroll
                    for (int i2 = 0; i2 < XW; ++i2) xb[k][i2] = xn[k][i2];
            }
        }
        // the largest weighted distance (non-negative doubles order like their bits)
        unsigned long long pb = (unsigned long long)__double_as_longlong(W ? pmax : (double)__uint_as_float(fmx));
        pb = wave_max_u64(pb);
        if (lane == 0) wave_max[wave] = pb;
        __syncthreads();
        unsigned long long pm = 0;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) pm = wave_max[w] > pm ? wave_max[w] : pm;
        if (pm == 0ull) {                                    // every token sits on a centre already
            if (tid == 0) pick_sh = (int)__umul64hi(rnd[j + 1], (unsigned long long)n);
            __syncthreads();
            continue;
        }
        const int kq = __builtin_amdgcn_readfirstlane(62 - log2n - ((int)((pm >> 52) & 0x7ffull) - 1023 + 1));
        draw(rnd[j + 1], kq);
    }
}

// ------------------------------------------------------------------------------------------
// Lloyd iteration
// ------------------------------------------------------------------------------------------
template <int C>
__global__ __launch_bounds__(kAssignThreads) void kmeans_assign_kernel(const uint16_t* xg_all, const float* cent_all,
                                                                      uint16_t* assign_all, int n, int K)
{
    extern __shared__ float cs[];                   // [K][C]
    const int g = blockIdx.y, tid = threadIdx.x;
    const float* cent = cent_all + (size_t)g * K * C;
    for (int i = tid; i < K * C; i += kAssignThreads) cs[i] = cent[i];
    __syncthreads();

    const uint16_t* xg = xg_all + (size_t)g * n * C;
    const int base = blockIdx.x * (kAssignThreads * kAssignPoints) + tid;
    float x[kAssignPoints][C];
    float best[kAssignPoints];
    int arg[kAssignPoints];
#pragma unroll
    for (int p = 0; p < kAssignPoints; ++p) {
        const int i = min(base + p * kAssignThreads, n - 1);
        widen<C>(xg + (size_t)i * C, x[p]);
        best[p] = dist2<C>(x[p], cs);
        arg[p] = 0;
    }
    for (int k = 1; k < K; ++k) {
        float c[C];
#pragma unroll
        for (int i = 0; i < C; ++i) c[i] = cs[k * C + i];
#pragma unroll
        for (int p = 0; p < kAssignPoints; ++p) {
            const float d = dist2<C>(x[p], c);
            arg[p] = d < best[p] ? k : arg[p];
            best[p] = d < best[p] ? d : best[p];
        }
    }
#pragma unroll
    for (int p = 0; p < kAssignPoints; ++p) {
        const int i = base + p * kAssignThreads;
        if (i < n) assign_all[(size_t)g * n + i] = (uint16_t)arg[p];
    }
}

// One workgroup: clusters [k0, k0 + 256) of one group.  Exact integer sums in LDS, then the new
// centroids of the clusters that own tokens.
template <int C>
__global__ __launch_bounds__(256) void kmeans_update_kernel(const uint16_t* xg_all, const uint32_t* wq_all,
                                                            const uint16_t* assign_all, float* cent_all, int n, int K)
{
    __shared__ unsigned long long s_hi[kUpdateClusters * C], s_lo[kUpdateClusters * C], wsum[kUpdateClusters];
    const int g = blockIdx.x, k0 = blockIdx.y * kUpdateClusters, tid = threadIdx.x;
    for (int i = tid; i < kUpdateClusters * C; i += 256) { s_hi[i] = 0ull; s_lo[i] = 0ull; }
    for (int i = tid; i < kUpdateClusters; i += 256) wsum[i] = 0ull;
    __syncthreads();
    const uint16_t* xg = xg_all + (size_t)g * n * C;
    const uint32_t* wq = wq_all + (size_t)g * n;
    const uint16_t* assign = assign_all + (size_t)g * n;
    for (int i = tid; i < n; i += 256) {
        const int k = (int)assign[i] - k0;
        if (k < 0 || k >= kUpdateClusters) continue;
        const long long w = (long long)wq[i];
        float xi[C];
        widen<C>(xg + (size_t)i * C, xi);
#pragma unroll
        for (int ch = 0; ch < C; ++ch) {
            const long long xq = (long long)ldexpf(xi[ch], 24);          // an integer: exact
            const long long hi = xq >> 20;                               // floor
            const long long lo = xq - hi * 1048576;
            atomicAdd(&s_hi[k * C + ch], (unsigned long long)(w * hi));
            atomicAdd(&s_lo[k * C + ch], (unsigned long long)(w * lo));
        }
        atomicAdd(&wsum[k], (unsigned long long)w);
    }
    __syncthreads();
    for (int e = tid; e < kUpdateClusters * C; e += 256) {
        const int k = e / C;
        if (k0 + k >= K) continue;
        const long long wk = (long long)wsum[k];
        if (wk == 0) continue;                      // a cluster without tokens keeps its centroid
        cent_all[((size_t)g * K + k0) * C + e] = kmeans_mean((long long)s_hi[e], (long long)s_lo[e], wk);
    }
}

__global__ void kmeans_finish_kernel(const float* cent, size_t count, uint16_t* out16, float* out32)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float v = cent[i];
    if (out16) out16[i] = __builtin_bit_cast(uint16_t, (_Float16)v);     // round to nearest even
    if (out32) out32[i] = v;
}

__global__ void kmeans_copy_u16_kernel(const uint16_t* src, uint16_t* dst, size_t count)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dst[i] = src[i];
}

__global__ void kmeans_copy_f32_kernel(const float* src, float* dst, size_t count)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dst[i] = src[i];
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int ceil_log2(int n)
{
    int l = 0;
    while ((1ll << l) < n) ++l;
    return l;
}

bool launch_ok() { return hipGetLastError() == hipSuccess; }

template <int C>
cq_status run_init(const KMeansArgs& a, const KMeansWorkspace& ws, hipStream_t st)
{
    const int G = a.f.groups, K = a.f.k, n = a.n;
    if (a.weights) {
        hipLaunchKernelGGL(kmeans_clear_kernel, dim3((G + 255) / 256), dim3(256), 0, st, ws.wmax_bits, G);
        const int rows = n < 256 ? n : 256;
        hipLaunchKernelGGL(kmeans_wmax_kernel, dim3((G + 255) / 256, rows), dim3(256), 0, st, a.weights, n, G, ws.wmax_bits);
    }
    hipLaunchKernelGGL((kmeans_prepare_kernel<C>), dim3((n + kPrepTokens - 1) / kPrepTokens, (G + kPrepGroups - 1) / kPrepGroups), dim3(256), 0, st, a.x, a.x_row_stride,
                       a.weights, ws.wmax_bits, n, G, ws.xg, ws.wq);
    if (!launch_ok()) return CQ_ERR_HIP;
    (void)K;
    return CQ_OK;
}

template <int C, bool W, int R>
cq_status launch_kmeanspp_resident(const KMeansArgs& a, const KMeansWorkspace& ws, hipStream_t st)
{
    auto kernel = kmeanspp_resident_kernel<C, W, R>;
    constexpr size_t lds = (size_t)kPPLdsRounds<C, W, R> * kPPThreads * C * 2 + (kPPWeightsInLds<W, R> ? (size_t)R * kPPThreads * 4 : 0) +
                           (2 * (kPPThreads / 64) + 1) * sizeof(uint64_t);
    static_assert(lds <= 160 * 1024, "one workgroup's LDS");
    static LdsKernelSetup setup;
    if (setup.ensure(reinterpret_cast<const void*>(kernel)) != hipSuccess) return CQ_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3(a.f.groups), dim3(kPPThreads), lds, st, ws.xg, ws.wq, a.rnd, a.picks, ws.cent, a.n, a.f.k,
                       ceil_log2(a.n));
    return launch_ok() ? CQ_OK : CQ_ERR_HIP;
}

// rounds of 1024 tokens: the smallest of the six unrolled forms that holds the call's tokens
template <int C, bool W>
cq_status launch_kmeanspp_rounds(const KMeansArgs& a, const KMeansWorkspace& ws, hipStream_t st)
{
    if (a.n <= kPPThreads) return launch_kmeanspp_resident<C, W, 1>(a, ws, st);
    if (a.n <= kPPThreads * 2) return launch_kmeanspp_resident<C, W, 2>(a, ws, st);
    if (a.n <= kPPThreads * 4) return launch_kmeanspp_resident<C, W, 4>(a, ws, st);
    if (a.n <= kPPThreads * 8) return launch_kmeanspp_resident<C, W, 8>(a, ws, st);
    if (a.n <= kPPThreads * 16) return launch_kmeanspp_resident<C, W, 16>(a, ws, st);
    return launch_kmeanspp_resident<C, W, kPPRounds>(a, ws, st);
}

template <int C>
cq_status run_kmeanspp(const KMeansArgs& a, const KMeansWorkspace& ws, hipStream_t st)
{
    if constexpr (C >= 2) {
        // The tokens' distances fit the registers of one workgroup.  Up to 128 tokens of groups that all run at once, one
        // per CU, the general kernel's picks wait for fewer barriers' worth of idle wavefronts (8 channels, 16 groups,
        // general / resident: 1 token 395 / 518 us, 64 484 / 556, 100 550 / 577, 128 586 / 592, 160 640 / 611); of more groups
        // two share a CU here and not there (512 groups, 100 tokens: 1096 / 885).
        const bool few = a.n <= 128 && a.f.groups <= 256;
        if (!few && a.n <= kPPThreads * kPPRounds) {
            return a.weights ? launch_kmeanspp_rounds<C, true>(a, ws, st) : launch_kmeanspp_rounds<C, false>(a, ws, st);
        }
    }
    hipLaunchKernelGGL((kmeanspp_kernel<C>), dim3(a.f.groups), dim3(kPPThreads), 0, st, ws.xg, ws.wq, ws.dmin, a.rnd, a.picks,
                       ws.cent, a.n, a.f.k, ceil_log2(a.n));
    return launch_ok() ? CQ_OK : CQ_ERR_HIP;
}

template <int C>
cq_status run_lloyd(const KMeansArgs& a, const KMeansWorkspace& ws, hipStream_t st)
{
    const int G = a.f.groups, K = a.f.k, n = a.n;
    if constexpr (C >= 2) {
        if (K == 256) {
            // the nearest-centre distances are done with, and the assignment goes to the caller: their room holds the
            // sums of token splits, with the weights' in front of it where all are one
            KMeansLloyd l;
            l.xg = ws.xg;
            l.wq = a.weights ? ws.wq : nullptr;
            l.cent = ws.cent;
            l.assign = a.assign_out;
            l.scratch = a.weights ? static_cast<void*>(ws.dmin) : ws.wq;
            l.scratch_bytes = (size_t)(reinterpret_cast<char*>(ws.assign + (size_t)G * n) - static_cast<char*>(l.scratch));
            l.groups = G;
            l.n = n;
            l.n_iter = a.n_iter;
            return launch_kmeans_lloyd(l, C, st);
        }
    }
    const size_t lds = sizeof(float) * (size_t)K * C;
    const dim3 agrid((n + kAssignThreads * kAssignPoints - 1) / (kAssignThreads * kAssignPoints), G);
    const dim3 ugrid(G, (K + kUpdateClusters - 1) / kUpdateClusters);
    for (int it = 0; it < a.n_iter; ++it) {
        hipLaunchKernelGGL((kmeans_assign_kernel<C>), agrid, dim3(kAssignThreads), lds, st, ws.xg, ws.cent, ws.assign, n, K);
        hipLaunchKernelGGL((kmeans_update_kernel<C>), ugrid, dim3(256), 0, st, ws.xg, ws.wq, ws.assign, ws.cent, n, K);
    }
    return launch_ok() ? CQ_OK : CQ_ERR_HIP;
}

template <int C>
cq_status run_all(const KMeansArgs& a, const KMeansWorkspace& ws, hipStream_t st)
{
    cq_status s = run_init<C>(a, ws, st);
    if (s != CQ_OK) return s;
    if (a.do_init) {
        s = run_kmeanspp<C>(a, ws, st);
        if (s != CQ_OK) return s;
    } else {
        const size_t cnt = (size_t)a.f.groups * a.f.k * C;
        hipLaunchKernelGGL(kmeans_copy_f32_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, a.cent_in, ws.cent, cnt);
    }
    s = run_lloyd<C>(a, ws, st);
    if (s != CQ_OK) return s;
    const size_t cnt = (size_t)a.f.groups * a.f.k * C;
    hipLaunchKernelGGL(kmeans_finish_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, ws.cent, cnt, a.cent16_out,
                       a.cent32_out);
    if (a.assign_out && a.n_iter > 0 && !(C >= 2 && a.f.k == 256)) {     // (the matrix-core iteration writes it itself)
        const size_t an = (size_t)a.f.groups * a.n;
        hipLaunchKernelGGL(kmeans_copy_u16_kernel, dim3((unsigned)((an + 255) / 256)), dim3(256), 0, st, ws.assign, a.assign_out, an);
    }
    return launch_ok() ? CQ_OK : CQ_ERR_HIP;
}

}  // namespace

size_t kmeans_workspace_layout(const Derived& f, int n, void* base, KMeansWorkspace* ws)
{
    const size_t G = (size_t)f.groups, K = (size_t)f.k, C = (size_t)f.c;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align256(off + bytes);
        return at;
    };
    const size_t o_xg = take(G * n * C * 2);
    const size_t o_wq = take(G * n * 4);
    const size_t o_dmin = take(G * n * 4);
    const size_t o_assign = take(G * n * 2);
    const size_t o_cent = take(G * K * C * 4);
    const size_t o_wmax = take(G * 4);
    if (ws) {
        char* b = static_cast<char*>(base);
        ws->xg = reinterpret_cast<uint16_t*>(b + o_xg);
        ws->wq = reinterpret_cast<uint32_t*>(b + o_wq);
        ws->dmin = reinterpret_cast<float*>(b + o_dmin);
        ws->assign = reinterpret_cast<uint16_t*>(b + o_assign);
        ws->cent = reinterpret_cast<float*>(b + o_cent);
        ws->wmax_bits = reinterpret_cast<unsigned*>(b + o_wmax);
    }
    return off;
}

cq_status launch_kmeans(const KMeansArgs& a, void* workspace, hipStream_t stream)
{
    KMeansWorkspace ws;
    kmeans_workspace_layout(a.f, a.n, workspace, &ws);
    switch (a.f.c) {
    case 8: return run_all<8>(a, ws, stream);
    case 4: return run_all<4>(a, ws, stream);
    case 2: return run_all<2>(a, ws, stream);
    case 1: return run_all<1>(a, ws, stream);
    default: return CQ_ERR_UNSUPPORTED;
    }
}

}  // namespace cq
