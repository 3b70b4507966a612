// Value codebooks in LDS as operands of matrix products: which codes of a 64-token tile a lane needs,
// where their entries are, and the read that gathers and transposes them.  Shared by the kernels
// that keep a KV head's codebooks on chip (cq_chunk_lds.hip, cq_decode_quad.hip).
#pragma once

#include "cq_decode_common.hpp"

namespace cq {
namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef short short4_t __attribute__((ext_vector_type(4)));

constexpr unsigned kBookBytes = 64 * 1024;              // one codebook of a KV head (CQ-8c8b, CQ-4c8b)

// lanes 16 b .. 16 b + 15 give the addresses of 4 rows of 16 fp16 numbers (lane 4 k + j: numbers 4 j .. 4 j + 3
// of row k); lane 16 b + j receives number j of the four rows
__device__ __forceinline__ half4_t lds_transposed(unsigned a)
{
    return __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_t*)(a)));
}
// The codes of one token that a lane needs, out of the token's record (byte w of plane p is slot
// 16 p + w, holding the code of group (slot + token) mod Gh): every STRIDE-th group from group
// g0 on, N of them, in group order, one byte each.  All of a lane's tokens are equal mod 16, and
// (Gh = 32) a pair of token blocks differs by 16, which is a rotation by 16 slots, i.e. the planes
// change places.
template <int GH, int STRIDE>
struct CodePick {
    static constexpr int N = GH / STRIDE;               // 4 or 8
    static constexpr int PL = GH / 16;
    unsigned sel0, sel1;                                // byte selectors of v_perm_b32
    unsigned rot;                                       // elements to rotate by
    bool swap;
    __device__ __forceinline__ CodePick(int g0, int token)
    {
        const unsigned beta = (unsigned)(g0 - token) & (GH - 1);
        if constexpr (STRIDE == 4) {
            const unsigned p = beta & 3;                // one byte of every dword
            sel0 = 0x0c0c0000u | p | ((4 + p) << 8);
            sel1 = 0x00000c0cu | (p << 16) | ((4 + p) << 24);
            rot = (beta >> 2) & 3;
            swap = (beta >> 2) >= 4;
        } else {
            const unsigned p = beta & 1;                // two bytes of every dword
            sel0 = p | ((p + 2) << 8) | ((p + 4) << 16) | ((p + 6) << 24);
            sel1 = 0;
            rot = (beta >> 1) & 3;
            swap = (beta >> 1) >= 4;
        }
    }
    __device__ __forceinline__ unsigned four(const u32x4& r) const
    {
        return __builtin_amdgcn_perm(r[1], r[0], sel0) | __builtin_amdgcn_perm(r[3], r[2], sel1);
    }
    // the N codes, four to a word, of a token in an even (odd = 0) or odd block of 16
    __device__ __forceinline__ void operator()(const u32x4 (&rec)[PL], int odd, unsigned (&z)[N / 4]) const
    {
        if constexpr (N == 4) {
            const unsigned x = four(rec[0]);
            z[0] = __builtin_amdgcn_alignbyte(x, x, rot);
        } else {
            unsigned x0, x1;
            if constexpr (STRIDE == 4) {
                x0 = four(rec[odd ? PL - 1 : 0]);
                x1 = four(rec[odd ? 0 : PL - 1]);
            } else {
                x0 = __builtin_amdgcn_perm(rec[0][1], rec[0][0], sel0);
                x1 = __builtin_amdgcn_perm(rec[0][3], rec[0][2], sel0);
            }
            const unsigned y0 = swap ? x1 : x0, y1 = swap ? x0 : x1;
            z[0] = __builtin_amdgcn_alignbyte(y1, y0, rot);
            z[1] = __builtin_amdgcn_alignbyte(y0, y1, rot);
        }
    }
};

// Whether a score of some query of this wavefront could reach `limit` (wavefront-uniform): |q|^2 <= q2, and a key of
// 128 channels is no longer than 65504 sqrt(128).  Scores that cannot are scaled inside the exponent of the
// probability, fma(x, scale, -ref); others before their maximum is taken: in the exponent, half a unit of a large
// score could carry the largest probability out of fp16's range.
__device__ __forceinline__ bool scores_may_be_large(float q2, float scale, float limit)
{
    const float l = limit / 65504.f;
    return __builtin_amdgcn_ballot_w64(!(q2 * (scale * scale) < l * l / 128.f)) != 0;
}

// LDS address of the entry of code byte k of z: code x entry size + `base`, the lane's part (codebook,
// first group, half), in one instruction (a dot product of bytes; shift, mask and or took two or three)
template <int C>
__device__ __forceinline__ unsigned entry(unsigned z, int k, unsigned base)
{
    return __builtin_amdgcn_udot4(z, (2u * C) << (8 * k), base, false);
}

template <int ABID>
__device__ __forceinline__ float4_t mfma_heads(half4_t q, half4_t k, float4_t c)
{
    return __builtin_amdgcn_mfma_f32_4x4x4f16(q, k, c, 4, ABID, 0);
}
// c += (channels 4 i .. 4 i + 3 of the four queries, from block i % 16 of register i / 16) x (those of the lane's key)
__device__ __forceinline__ float4_t mfma_quad(const half4_t (&q)[2], half4_t k, float4_t c, int i)
{
    const half4_t a = q[i >> 4];
    switch (i & 15) {
        case 0: return mfma_heads<0>(a, k, c);
        case 1: return mfma_heads<1>(a, k, c);
        case 2: return mfma_heads<2>(a, k, c);
        case 3: return mfma_heads<3>(a, k, c);
        case 4: return mfma_heads<4>(a, k, c);
        case 5: return mfma_heads<5>(a, k, c);
        case 6: return mfma_heads<6>(a, k, c);
        case 7: return mfma_heads<7>(a, k, c);
        case 8: return mfma_heads<8>(a, k, c);
        case 9: return mfma_heads<9>(a, k, c);
        case 10: return mfma_heads<10>(a, k, c);
        case 11: return mfma_heads<11>(a, k, c);
        case 12: return mfma_heads<12>(a, k, c);
        case 13: return mfma_heads<13>(a, k, c);
        case 14: return mfma_heads<14>(a, k, c);
        default: return mfma_heads<15>(a, k, c);
    }
}

}  // namespace
}  // namespace cq
