// Device code shared by the k-means kernels (cq_kmeans.hip, cq_kmeans_mfma.hip): the arithmetic that
// decides an assignment.  Internal linkage: every translation unit gets its own copy.
#pragma once

#include <hip/hip_runtime.h>

#include "cq_internal.hpp"

namespace cq {
namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

template <int C>
__device__ __forceinline__ void widen(const uint16_t* p, float (&v)[C])
{
    if constexpr (C == 8) {
        const uint4 a = *reinterpret_cast<const uint4*>(p);
        const unsigned w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const half2_t h = __builtin_bit_cast(half2_t, w[i]);
            v[2 * i] = (float)h.x;
            v[2 * i + 1] = (float)h.y;
        }
    } else if constexpr (C == 4) {
        const uint2 a = *reinterpret_cast<const uint2*>(p);
        const half2_t h0 = __builtin_bit_cast(half2_t, a.x), h1 = __builtin_bit_cast(half2_t, a.y);
        v[0] = (float)h0.x; v[1] = (float)h0.y; v[2] = (float)h1.x; v[3] = (float)h1.y;
    } else if constexpr (C == 2) {
        const half2_t h = __builtin_bit_cast(half2_t, *reinterpret_cast<const unsigned*>(p));
        v[0] = (float)h.x; v[1] = (float)h.y;
    } else {
        static_assert(C == 1, "channels per group: 1, 2, 4 or 8");
        v[0] = (float)__builtin_bit_cast(_Float16, *p);
    }
}

template <int C>
__device__ __forceinline__ float dist2(const float (&x)[C], const float* c)
{
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const float d = x[i] - c[i];
        acc = __builtin_fmaf(d, d, acc);
    }
    return acc;
}

// The new coordinate of a cluster from its exact sums: weighted sums of floor(16 x) and of the rest in
// units of 2^-24 (S = hi 2^20 + lo) over the sum of the weights; or S itself (weights of one: hi 2^20
// and lo are then both exact in fp64, so their sum rounds like S).
__device__ __forceinline__ float kmeans_mean(long long hi, long long lo, long long w)
{
    const double num = (double)hi * 1048576.0 + (double)lo;
    return (float)(num / (double)w * 0x1p-24);
}
__device__ __forceinline__ float kmeans_mean(long long sum, long long w) { return (float)((double)sum / (double)w * 0x1p-24); }

}  // namespace
}  // namespace cq
