// Device code shared by the two kernels of decode attention over keys as stored (cq_decode.hip: a query head per
// workgroup; cq_decode_pair.hip: two): partials and their merge, the new token's record, a tile's request.
#pragma once

#include "cq_decode_common.hpp"

namespace cq {
namespace {

constexpr int kDecodeThreads = 512;
constexpr int kDecodeWaves = kDecodeThreads / 64;
// tiles per wavefront and chunk (= score registers per lane): b = 8: 16, and 8 for splits that fit;
// b = 10: 32 (one chunk must hold the longest split, 16384 tokens), and 16 for splits that fit
constexpr int kChunkTiles8 = 16;
constexpr int kChunkTiles10 = 32;

// LayerPtrs as the kernel reads it.  A pointer read from memory could point anywhere (LDS,
// scratch) as far as the compiler knows, and every access through it would be a flat instruction,
// which waits on the LDS counter and the memory counter at once; the table's pointers are
// therefore declared as what they are, pointers into global memory.
#define CQ_GLOBAL __attribute__((address_space(1)))
struct LayerPtrsGlobal {
    CQ_GLOBAL const uint16_t* q;
    CQ_GLOBAL const uint16_t* xk_new;
    CQ_GLOBAL const uint16_t* xv_new;
    CQ_GLOBAL uint8_t* k_codes;
    CQ_GLOBAL uint8_t* v_codes;
    CQ_GLOBAL const uint16_t* k_centroids;
    CQ_GLOBAL const uint16_t* v_centroids;
    CQ_GLOBAL uint16_t* out;
};
#undef CQ_GLOBAL
static_assert(sizeof(LayerPtrsGlobal) == sizeof(LayerPtrs), "same record");

// Merge the partials of all splits of one (sequence, query head): one pass with a running
// maximum (the usual rescaling), so that no load waits for a value computed from another and
// the loads of all splits go out together; then one rounding to fp16.  A split beyond its
// sequence left m = -inf, l = 0, o = 0 and gets weight 0.  DEVICE_LOADS: the partials were
// written by other workgroups of the running kernel: read them with device-scope loads.
template <bool DEVICE_LOADS>
__device__ __forceinline__ float partial_load(const float* p)
{
    if constexpr (DEVICE_LOADS) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}
template <bool DEVICE_LOADS>
__device__ __forceinline__ void merge_splits(const float* p, int n_split, int head_dim, uint16_t* out, int tid, int nt)
{
    const int stride = head_dim + kPartialHeader;
    for (int i = tid; i < head_dim; i += nt) {
        float m = -INFINITY, l = 0.f, o = 0.f;
#pragma unroll 4
        for (int s = 0; s < n_split; ++s) {
            const float ms = partial_load<DEVICE_LOADS>(p + s * stride), ls = partial_load<DEVICE_LOADS>(p + s * stride + 1),
                        os = partial_load<DEVICE_LOADS>(p + s * stride + kPartialHeader + i);
            const float m_new = fmaxf(m, ms);
            const float m_safe = m_new == -INFINITY ? 0.f : m_new;
            const float keep = __builtin_amdgcn_exp2f(m - m_safe), w = __builtin_amdgcn_exp2f(ms - m_safe);
            l = __builtin_fmaf(l, keep, ls * w);
            o = __builtin_fmaf(o, keep, os * w);
            m = m_new;
        }
        const _Float16 h = (_Float16)(o / l);
        out[i] = __builtin_bit_cast(uint16_t, h);
    }
}
// (device-scope store: written through to where every workgroup's device-scope loads find it)
__device__ __forceinline__ void partial_store(float* p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The last split of a (sequence, query head) to finish merges them all.  Partials are written with device-scope
// stores (write-through) and the merging workgroup reads them with device-scope loads, so
// no cache has to be written back or invalidated as a whole (a device-scope release fence
// per workgroup, which writes the whole L2 back, cost 50 us on a 90 us launch).  Order:
// every wavefront waits for its stores (a barrier does not, __syncthreads() neither), then all meet at the
// barrier, then one thread counts the workgroup in; the workgroup that counts the last split (true) takes the counter
// back to zero for the next call.
template <int D>
__device__ __forceinline__ bool counted_last(const DecodeArgs& a, const float* part, unsigned* flag, int tid)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        const size_t row = (size_t)(part - a.partials) / ((size_t)(D + kPartialHeader) * a.n_split);
        const unsigned arrived = __hip_atomic_fetch_add(a.merge_counters + row, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool last = arrived == (unsigned)a.n_split - 1u;
        if (last) __hip_atomic_store(a.merge_counters + row, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = last;
    }
    __syncthreads();
    return *flag != 0u;
}

// Fused step: words of LDS from the keys on.  The 2 Gh 64-bit minima; the new token's fixed-point weight, one per query
// head of the workgroup, in 16 bytes; the record of its key codes (NewTokenRecord), read 16 bytes at a time.
template <int GH, int B>
struct NewTokenWords {
    static constexpr int WEIGHT = 2 * 2 * GH;
    static constexpr int RECORD = WEIGHT + 4;
    static constexpr int END = RECORD + GH / 4 + (B == 10 ? 1 : 0);
};

// Fused step: the key codes of the new token as the cache layout would hold them (slot s of token
// u carries group (s + u) mod Gh), from keys[g] = group g's (distance, index) minimum.  Built in LDS
// by the one wavefront whose walk meets the token's tile, before its walk starts (lane i builds word
// i); when the walk reaches the tile, lane u's codes are replaced by the record.
template <int GH, int B>
struct NewTokenRecord {
    unsigned* rec;                      // [GH / 4] words of low bytes, then (b = 10) the word of high bits
    __device__ __forceinline__ void build(const unsigned long long* keys, int u_new, int lane) const
    {
        unsigned x = 0, h = 0;
        if (lane < GH / 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int s = 4 * lane + k;
                const unsigned code = (unsigned)(keys[(s + u_new) & (GH - 1)] & 0xffffffffu);
                x |= (code & 0xffu) << (8 * k);
                if constexpr (B == 10) h |= (code >> 8) << (2 * s);
            }
            rec[lane] = x;
        }
        if constexpr (B == 10) {
            static_assert(B != 10 || GH == 16, "four lanes hold the high bits");
            h |= __shfl_xor(h, 1);
            h |= __shfl_xor(h, 2);
            if (lane == 0) rec[GH / 4] = h;
        }
    }
    __device__ __forceinline__ void patch(Tile<GH, B>& w, int u_new, int lane) const
    {
        const bool mine = lane == u_new;
#pragma unroll
        for (int pl = 0; pl < GH / 16; ++pl) {
            const uint4 r = *reinterpret_cast<const uint4*>(rec + 4 * pl);
            u32x4 q = w.lo[pl];
            q.x = mine ? r.x : q.x;
            q.y = mine ? r.y : q.y;
            q.z = mine ? r.z : q.z;
            q.w = mine ? r.w : q.w;
            w.lo[pl] = q;
        }
        if constexpr (B == 10) w.hi = mine ? rec[GH / 4] : w.hi;
    }
};

// One 64-token tile through a buffer descriptor of its own: `tile` is wave-uniform; a tile that
// does not exist gets a descriptor of size zero, for which the hardware returns zeros without
// touching memory.  Every request of the walk is therefore issued unconditionally, and the
// number of loads in flight at any point of the (unrolled) walk is a compile-time constant.
template <int GH, int B>
__device__ __forceinline__ Tile<GH, B> load_tile_desc(const uint8_t* tile, bool exists, int lane)
{
    constexpr int TB = kTileTokens * GH * B / 8;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(tile), 0, exists ? TB : 0, 0x00020000);
    Tile<GH, B> w;
    const unsigned off = 16u * (unsigned)lane;
#pragma unroll
    for (int pl = 0; pl < GH / 16; ++pl)
        w.lo[pl] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + 1024u * pl, 0, 2));
    if constexpr (B == 10)
        w.hi = __builtin_amdgcn_raw_buffer_load_b32(rsrc, 4u * (unsigned)lane + (unsigned)(kTileTokens * GH), 0, 2);
    else
        w.hi = 0;
    return w;
}

}  // namespace
}  // namespace cq
