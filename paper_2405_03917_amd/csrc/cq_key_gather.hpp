// Keys by code, one token per lane: the token's codes in group order, a centroid out of LDS, its rotation by the
// lane's part of a position, and the products that sum over channels for four query heads at once.  Shared by the
// kernels that read key centroids from LDS (cq_decode_rope.hip, cq_decode_quad.hip).
#pragma once

#include "cq_decode_common.hpp"

namespace cq {
namespace {

constexpr int kPairs = 64;                        // head_dim / 2
// The softmax reference of a head or row that has seen no token.  Finite: tokens that score -inf (masked, or beyond the
// range of fp32) then have weight 2^-inf = 0, where a reference of -inf gives 2^(-inf + inf).
constexpr float kNoScore = -3.0e38f;

template <int C>
struct CenVec {
    unsigned w[C / 2];
};
template <int C>
__device__ __forceinline__ CenVec<C> lds_centroid(unsigned byte_addr)
{
    typedef __attribute__((address_space(3))) unsigned lds_u;
    CenVec<C> v;
    if constexpr (C == 8) {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const u4 a = *(__attribute__((address_space(3))) u4*)(byte_addr);
        v.w[0] = a.x; v.w[1] = a.y; v.w[2] = a.z; v.w[3] = a.w;
    } else if constexpr (C == 4) {
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        const u2 a = *(__attribute__((address_space(3))) u2*)(byte_addr);
        v.w[0] = a.x; v.w[1] = a.y;
    } else {
        v.w[0] = *(lds_u*)(byte_addr);
    }
    return v;
}
// A token's codes in group order.  The cache stores the code of group (s + u) mod Gh in slot s
// of token u (the position-independent kernel wants neighbouring lanes on different groups);
// here every lane should work on the same channel pair at the same time (the rotated query is
// then a scalar, and every table address a compile-time offset), so the token's Gh bytes are
// rotated by u positions once per tile: bytes first (v_alignbyte), then whole dwords (selects).
struct Unrotate {
    unsigned bytes;             // (Gh - u) mod 4
    unsigned dwords;            // ((Gh - u) mod Gh) / 4
};
template <int GH, int B>
__device__ __forceinline__ void group_order(const Tile<GH, B>& w, const Unrotate& r, unsigned (&d)[GH / 4])
{
    constexpr int N = GH / 4;
    unsigned x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const u32x4 q = w.lo[i >> 2];
        x[i] = (i & 3) == 0 ? q.x : (i & 3) == 1 ? q.y : (i & 3) == 2 ? q.z : q.w;
    }
    // group g sits in slot (g - u) mod Gh = (g + r) mod Gh with r = (Gh - u) mod Gh
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = __builtin_amdgcn_alignbyte(x[(i + 1) % N], x[i], r.bytes);
#pragma unroll
    for (int bit = 1; bit < N; bit <<= 1) {
        const bool on = (r.dwords & bit) != 0;
        unsigned y[N];
#pragma unroll
        for (int i = 0; i < N; ++i) y[i] = on ? d[(i + bit) % N] : d[i];
#pragma unroll
        for (int i = 0; i < N; ++i) d[i] = y[i];
    }
}

// acc += (the query values of pair i, one head per row) x (the rotated key of pair i, one token per
// column): the A operand is register i / 16 of the per-tile query registers, broadcast from the
// block of four lanes i % 16.
typedef float mfma_f4 __attribute__((ext_vector_type(4)));
template <int ABID>
__device__ __forceinline__ mfma_f4 mfma_bcast(float a, float b, mfma_f4 c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, ABID, 0);
}
__device__ __forceinline__ mfma_f4 mfma_pair(const float (&q)[4], float x, mfma_f4 c, int i)
{
    const float a = q[i >> 4];
    switch (i & 15) {
        case 0: return mfma_bcast<0>(a, x, c);
        case 1: return mfma_bcast<1>(a, x, c);
        case 2: return mfma_bcast<2>(a, x, c);
        case 3: return mfma_bcast<3>(a, x, c);
        case 4: return mfma_bcast<4>(a, x, c);
        case 5: return mfma_bcast<5>(a, x, c);
        case 6: return mfma_bcast<6>(a, x, c);
        case 7: return mfma_bcast<7>(a, x, c);
        case 8: return mfma_bcast<8>(a, x, c);
        case 9: return mfma_bcast<9>(a, x, c);
        case 10: return mfma_bcast<10>(a, x, c);
        case 11: return mfma_bcast<11>(a, x, c);
        case 12: return mfma_bcast<12>(a, x, c);
        case 13: return mfma_bcast<13>(a, x, c);
        case 14: return mfma_bcast<14>(a, x, c);
        default: return mfma_bcast<15>(a, x, c);
    }
}

// The mixed-precision multiply-adds with a vector operand in place of the scalar one.
__device__ __forceinline__ float mixv_mul(bool HI, unsigned w, float s)
{
    float d;
    if (HI) asm volatile("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(w), "v"(s));
    else asm volatile("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(w), "v"(s));
    return d;
}
// (Its result feeds a matrix instruction.  The compiler does not look inside an asm statement, so
// it cannot know that a vector instruction wrote the register and leaves out the two wait states
// that a matrix instruction reading it needs.  The caller keeps the two apart instead: all
// sixteen results of a batch pass through one more (empty) statement before the first matrix
// instruction may read any of them, so that at least eight instructions lie between a result
// and its use.)
template <bool MINUS>
__device__ __forceinline__ float mixv_fma(bool HI, unsigned w, float s, float c)
{
    float d;
    if (HI && MINUS) asm volatile("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(w), "v"(s), "v"(c));
    else if (HI) asm volatile("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(w), "v"(s), "v"(c));
    else if (MINUS) asm volatile("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(w), "v"(s), "v"(c));
    else asm volatile("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(w), "v"(s), "v"(c));
    return d;
}

}  // namespace
}  // namespace cq
