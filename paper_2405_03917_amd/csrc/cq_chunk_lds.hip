// Causal attention of a few query rows per KV head over a packed CQ cache (speculative
// verification, short prefill chunks), for gfx950: the codebooks of the KV head in LDS, every
// wavefront on tiles of its own.  The formats whose two codebooks fit there: CQ-8c8b and CQ-4c8b
// (2 x 64 KB of the CU's 160 KB).
//
// The kernel for many rows (cq_chunk.hip) expands each 64-token tile once per workgroup from
// codebooks in L2, which costs it 2 x 64 x Gh divergent lane-gathers of the texture path per
// tile (about 4100 clocks at CQ-4c8b) whatever the number of rows.  Here the expansion IS the
// operand load of the matrix product:
//   S^T = K Q^T      v_mfma_f32_16x16x32_f16, A = keys of 16 tokens: a lane's 8 channels are the
//                    centroid(s) of its token's code(s), read by ds_read_b128 / b64 at code
//                    times entry size; B = 16 query rows (registers)
//   softmax          each lane owns one query column; 2^12-scaled probabilities as two fp16
//                    numbers (22 bits) as in cq_chunk.hip
//   O^T += V^T P^T   A = values transposed: ds_read_b64_tr_b16 takes an address per lane and
//                    hands lane j of 16 the j-th of 16 channels of 4 tokens, so gather and
//                    transpose are one instruction; B = the probabilities just computed
// A tile costs a wavefront 48 (CQ-8c8b) or 64 (4c8b) LDS gathers, 48 matrix products (32 up to 8
// rows) and about 260 / 330 vector instructions, nothing is shared between wavefronts inside the
// loop and there is no barrier.  Bound: the LDS.  A gather of 64 random 16-byte entries takes
// 12.3 clocks (16 lanes at a time on 16 bank groups: the fullest holds 3.1), a transposing one
// 6.2, i.e. 394 clocks per tile and CU at CQ-8c8b; the kernel takes 488 (LDS active 79 %; up to eight rows).
// Measured: CQ-4c8b, batch 16, 32 heads, 5 tokens over 4096: 136 us token by token, 264 us in the
// many-row kernel, 43 to 49 us here; CQ-8c8b, batch 4 x 131072, 5 tokens: 441 -> 271 us in two pieces (given as
// tokens_per_split: the default's workspace holds one, and such a call goes token by token).  The first form
// waited for every gather by itself (5800 clocks per tile and wavefront, 61 us); values gathered
// ahead of the softmax in one batch of 64 registers spilled at CQ-4c8b and gained nothing.
//
// A workgroup of 8 wavefronts (one per CU) serves RB = 1, 2 or 4 blocks of 16 rows; the 8 / RB wavefronts of
// a block take every (8 / RB)-th tile and are merged through LDS at the end.  Workgroups walk
// several (sequence, split) items of one KV head, so the codebooks are staged once per workgroup.
// Parts, each taken out by itself (32 heads): all keys of a tile gathered at once and not two of four batches ahead, CQ-8c8b, 40 tokens, 64 x 1000
// 143.4 -> 140.3 us, 16 tokens 62.8 -> 61.5; CQ-4c8b, 5 tokens of 16 x 4096, 43.3 -> 42.9.  Priorities: CQ-8c8b, 40 tokens
// of 64 x 1000, 145.4 -> 140.3, CQ-4c8b, 5 tokens of 16 x 4096, 44.2 -> 42.9, of 64 x 300 44.8 -> 45.8; up to eight rows of CQ-8c8b do without
// (5 tokens of 64 x 1000 52.6, with them 55.7; 8 of 16 x 16384 119.0 and 123.8).  Codebooks ahead of the first codes and eight rows merged in one
// pass: the rest of CQ-8c8b, 5 tokens of 64 x 1000, 57.9 -> 52.6, 16 x 4096 39.2 -> 36.9.
#include "cq_key_gather.hpp"
#include "cq_lds_gather.hpp"

namespace cq {
namespace {

constexpr int kWaves = 8;
constexpr int kRows = 16;                               // query rows of a wavefront
constexpr unsigned kMergeBase = 2 * kBookBytes;         // (m, l) of every wavefront and row, or 64 channels of every wavefront's
constexpr unsigned kORow = 64 * 4;                      // output rows
constexpr unsigned kLdsBytes = kMergeBase + kWaves * kRows * kORow;
static_assert(kLdsBytes == 160 * 1024, "all of a CU's LDS");
__device__ __forceinline__ half8_t lds_half8(unsigned a) { return *(__attribute__((address_space(3))) half8_t*)(a); }
__device__ __forceinline__ half4_t lds_half4(unsigned a) { return *(__attribute__((address_space(3))) half4_t*)(a); }
// The exponent that probabilities are relative to where the largest score (base 2) is m: 12 below m, so that
// they fill fp16's range; m itself where 12 is lost in its rounding.
__device__ __forceinline__ float softmax_reference(float m) { return m - (fabsf(m) < 0x1p22f ? 12.f : 0.f); }
// maximum / sum over the four lanes l % 16 + 16 b
__device__ __forceinline__ float across_max(float v)
{
    return rows_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float across_sum(float v)
{
    return rows_reduce(v, [](float a, float b) { return a + b; });
}

// HALF: at most 8 rows in all.  Columns q and q + 8 of the score product hold the same query, and in the
// value product the high parts of its probabilities in one and the low parts in the other: half the
// matrix products there, one addition at the end.
template <int C, bool HALF>
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(kWaves * 64) void chunk_lds_kernel(ChunkArgs a, int rb_log2, int items)
{
    constexpr int D = 128;
    constexpr int GH = D / C;
    constexpr int PL = GH / 16;
    constexpr int TILE_BYTES = kTileTokens * GH;
    extern __shared__ float smem[];
    (void)smem;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, blk = lane >> 4;

    const int cs = kWaves >> rb_log2;                       // context slices of each of the 2^rb_log2 row blocks
    const int rb = wave >> (3 - rb_log2), slice = wave & (cs - 1);
    const int hkv = blockIdx.x % a.f.n_kv_heads;
    const int stride = gridDim.x / a.f.n_kv_heads;
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    const int rows_total = a.m * qper;

    // ---- this lane's places: keys, token col of a block of 16, groups blk, blk + 4, ...; values, token
    // 4 blk + col / 4 of a block, channels 4 (col % 4) .. of 16 (C = 8: half of group (col % 4) / 2, then
    // every second group; C = 4: group col % 4, then every fourth)
    const int vtok = 4 * blk + (col >> 2);
    const CodePick<GH, 4> kpick(blk, col);
    const CodePick<GH, C == 8 ? 2 : 4> vpick(C == 8 ? (col & 3) >> 1 : (col & 3), vtok);
    const unsigned kbase = (unsigned)blk * (256 * 2 * C);
    const unsigned vbase = kBookBytes + (C == 8 ? ((unsigned)(col & 3) >> 1) * 4096 + (unsigned)(col & 1) * 8 : (unsigned)(col & 3) * 2048);


    // ---- the items of this workgroup: (sequence, split), advanced without divisions
    const float inv_qper = 1.f / (float)qper;
    const auto row_token = [&](int row) { return (int)(((float)row + 0.5f) * inv_qper); };     // row / qper (few rows: exact)
    int item = blockIdx.x / a.f.n_kv_heads;
    int split = item % a.n_split, n = item / a.n_split;
    const int d_split = stride % a.n_split, d_n = stride / a.n_split;
    int row0 = rb * kRows;                                  // (a block beyond the last row repeats it and stores nothing)
    struct Item {
        int n, split, pos, pos_first, tile0, tile1;
    };
    // (a scale of zero stands for one so small that every weight is 1: 0 times a masked -infinity is no number)
    const float scale = a.scale_log2e == 0.f ? 1e-37f : fabsf(a.scale_log2e);
    half8_t qreg[4];
    // the records of a tile on their way from memory, and the codes of one that this lane needs
    u32x4 rk[4][PL], rv[4][PL];                             // token 16 i + col, token 16 i + vtok
    unsigned zk[4][GH / 16], zv[4][2];
    auto request = [&](const Item& it, int tile) {
        const size_t at = a.map.tile_index(it.n, hkv, max(min(tile, it.tile1 - 1), it.tile0)) * TILE_BYTES;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int p = 0; p < PL; ++p) {
                rk[i][p] = *reinterpret_cast<const u32x4*>(a.k_codes + at + p * 1024 + (16 * i + col) * 16);
                rv[i][p] = *reinterpret_cast<const u32x4*>(a.v_codes + at + p * 1024 + (16 * i + vtok) * 16);
            }
    };
    auto unpack = [&]() {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            kpick(rk[i], i & 1, zk[i]);
            vpick(rv[i], i & 1, zv[i]);
        }
    };
    // an item's places, its queries and its first tile's records (requested ahead of the codebooks or of
    // the previous item's merge)
    auto open_item = [&]() {
        // (opaque per item: what follows from it would be kept in registers through the tiles, which spill then)
        asm volatile("" : "+s"(row0));
        Item it;
        it.n = n;
        it.split = split;
        int t_n = a.t;
        if (a.seq_lens) t_n = min(max(a.seq_lens[n], a.m), a.t);
        const int pos0 = t_n - a.m;                         // position of query token 0
        const int row = min(row0 + (HALF ? col & 7 : col), rows_total - 1);
        const int j = row_token(row);
        it.pos = pos0 + j;
        it.pos_first = __builtin_amdgcn_readfirstlane(pos0 + row_token(min(row0, rows_total - 1)));
        const int last_row = min(row0 + kRows, rows_total) - 1;
        const int last_tile = __builtin_amdgcn_readfirstlane((pos0 + row_token(last_row)) / kTileTokens);
        it.tile0 = split * a.tiles_per_split;
        it.tile1 = row0 < rows_total ? min(it.tile0 + a.tiles_per_split, last_tile + 1) : it.tile0;
        const uint16_t* qrow = a.q + (((size_t)n * a.m + j) * a.n_q_heads + hkv * qper + (row - j * qper)) * D;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if constexpr (C == 8) {
                qreg[s] = *reinterpret_cast<const half8_t*>(qrow + 32 * s + 8 * blk);
            } else {
                const half4_t lo = *reinterpret_cast<const half4_t*>(qrow + 32 * s + 4 * blk);
                const half4_t hi = *reinterpret_cast<const half4_t*>(qrow + 32 * s + 16 + 4 * blk);
                qreg[s] = half8_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
        }
        request(it, it.tile0 + slice);
        return it;
    };
    // ---- both codebooks of the head to LDS as they are ([group][code] entries); requested ahead of the first codes, which
    // come from further away (loads return in order)
    typedef __attribute__((address_space(3))) u32x4 lds_q;
    u32x4 book[2][8];
    {
        const u32x4* src[2] = {reinterpret_cast<const u32x4*>(a.k_centroids + (size_t)hkv * GH * 256 * C),
                               reinterpret_cast<const u32x4*>(a.v_centroids + (size_t)hkv * GH * 256 * C)};
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll
            for (int i = 0; i < 8; ++i) book[w][i] = src[w][i * (kWaves * 64) + tid];
    }
    __builtin_amdgcn_sched_barrier(0);
    Item it = open_item();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int i = 0; i < 8; ++i) *(lds_q*)(w * kBookBytes + (unsigned)(i * (kWaves * 64) + tid) * 16) = book[w][i];

    lds_barrier();

#pragma unroll 1
    for (;;) {
        float4_t o[8];
#pragma unroll
        for (int cb = 0; cb < 8; ++cb) o[cb] = float4_t{0.f, 0.f, 0.f, 0.f};
        float ref = -INFINITY, l_run = 0.f;             // probabilities and their sum are relative to 2^ref

        // (a negative scale goes into the queries, so that the largest product is the largest score)
        if (a.scale_log2e < 0.f) {
#pragma unroll
            for (int s = 0; s < 4; ++s) qreg[s] = -qreg[s];
        }
        // (no element of Q Q^T is larger than the largest of its diagonal, the squares of the queries' norms)
        float4_t g = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) g = __builtin_amdgcn_mfma_f32_16x16x32_f16(qreg[s], qreg[s], g, 0, 0, 0);
        const bool large = scores_may_be_large(fmaxf(fmaxf(g[0], g[1]), fmaxf(g[2], g[3])), scale, 0x1p24f);
        int tile = it.tile0 + slice;
        unpack();
        request(it, tile + cs);
        const float mult = large ? 1.f : scale, early = large ? scale : 1.f;
        bool turn = wave < kWaves / 2;                  // (priorities as in cq_decode_quad.hip)
        constexpr bool kPriorities = !(HALF && C == 8);
#pragma unroll 1
        for (; tile < it.tile1; tile += cs) {
            // All keys of the tile are gathered at once, the values in batches that the products behind them work off, one batch
            // ahead (the scheduling fences pin that order: left alone, the compiler waits for every gather by itself,
            // 130 clocks each).
            // ---- scores: acc[i][e] is token 16 i + 4 blk + e, query col
            if constexpr (kPriorities) {
                turn = !turn;
                if (turn) __builtin_amdgcn_s_setprio(1);
                else __builtin_amdgcn_s_setprio(0);
            }
            float4_t acc[4];
            half8_t kv[4][4];
            auto gather_keys = [&](int i) {
                unsigned at[GH / 4];
#pragma unroll
                for (int k = 0; k < GH / 4; ++k) at[k] = entry<C>(zk[i][k >> 2], k & 3, kbase);
                __builtin_amdgcn_sched_barrier(0);          // (addresses first: a gather right behind its own would wait for it)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    if constexpr (C == 8) {
                        kv[i][s] = lds_half8(at[s] + (unsigned)s * 16384);
                    } else {
                        const half4_t lo = lds_half4(at[2 * s] + (unsigned)(2 * s) * 8192);
                        const half4_t hi = lds_half4(at[2 * s + 1] + (unsigned)(2 * s + 1) * 8192);
                        kv[i][s] = half8_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    }
                }
            };
            half8_t av[2][8];
            auto gather_values = [&](int t) {
                unsigned at[2][8];
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int cb = 0; cb < 8; ++cb) at[h][cb] = entry<C>(zv[2 * t + h][cb >> 2], cb & 3, vbase);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int cb = 0; cb < 8; ++cb) {
                    const half4_t v0 = lds_transposed(at[0][cb] + (unsigned)cb * 8192), v1 = lds_transposed(at[1][cb] + (unsigned)cb * 8192);
                    av[t][cb] = half8_t{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                }
            };
            gather_keys(0);
            gather_keys(1);
            gather_keys(2);
            gather_keys(3);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[i] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; ++s) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kv[i][s], qreg[s], acc[i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            gather_values(0);
            __builtin_amdgcn_sched_barrier(0);
            // ---- online softmax of the lane's query column
            if constexpr (kPriorities) {
                if (turn) __builtin_amdgcn_s_setprio(3);
                else __builtin_amdgcn_s_setprio(2);
            }
            if (large || tile * kTileTokens + kTileTokens - 1 > it.pos_first) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int tok = tile * kTileTokens + 16 * i + 4 * blk + e;
                        acc[i][e] = tok <= it.pos ? acc[i][e] * early : -INFINITY;
                    }
            }
            float bmax = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) bmax = fmaxf(bmax, acc[i][e]);
            const float ref_new = fmaxf(ref, softmax_reference(across_max(bmax) * mult));
            const float shift = ref_new == -INFINITY ? 0.f : ref_new;       // nothing visible yet: all weights 0
            const float alpha = __builtin_amdgcn_exp2f(ref - shift);
            ref = ref_new;
            float psum = 0.f;
            half8_t ph[2], pl[2];                           // p = ph + pl to 22 bits (HALF: ph of columns q, q + 8)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    const float2_t ps = {__builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][e], mult, -shift)),
                                         __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][e + 1], mult, -shift))};
                    psum += ps[0];
                    psum += ps[1];
                    const half2_t hi = __builtin_convertvector(ps, half2_t);
                    const float2_t rest = {__builtin_fmaf((float)hi[0], -1.f, ps[0]), __builtin_fmaf((float)hi[1], -1.f, ps[1])};
                    const half2_t lo = __builtin_convertvector(rest, half2_t);
                    const int at = 4 * (i & 1) + e;
                    if constexpr (HALF) {
                        const half2_t v = __builtin_bit_cast(half2_t, col < 8 ? __builtin_bit_cast(unsigned, hi) : __builtin_bit_cast(unsigned, lo));
                        ph[i >> 1][at] = v[0];
                        ph[i >> 1][at + 1] = v[1];
                    } else {
                        ph[i >> 1][at] = hi[0];
                        ph[i >> 1][at + 1] = hi[1];
                        pl[i >> 1][at] = lo[0];
                        pl[i >> 1][at + 1] = lo[1];
                    }
                }
            l_run = __builtin_fmaf(l_run, alpha, psum);
            if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
                for (int cb = 0; cb < 8; ++cb) o[cb] *= alpha;
            }
            // ---- O^T += V^T P^T: contraction index (blk, 4 h + e) is token 32 t + 16 h + 4 blk + e
            __builtin_amdgcn_sched_barrier(0);
            gather_values(1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int cb = 0; cb < 8; ++cb) {
                    o[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[t][cb], ph[t], o[cb], 0, 0, 0);
                    if constexpr (!HALF) o[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[t][cb], pl[t], o[cb], 0, 0, 0);
                }
            // the next tile's codes, and the request for the tile after it
            unpack();
            request(it, tile + 2 * cs);
        }

        // ---- the next item's requests go out, then the context slices of every row block are merged: (ref, l),
        // then the rows, scaled to the common maximum, 64 channels at a time
        const Item done = it;
        item += stride;
        const bool more = item < items;
        if (more) {
            split += d_split;
            const int c1 = split >= a.n_split;
            split -= c1 ? a.n_split : 0;
            n += d_n + c1;
            it = open_item();
        }
        typedef __attribute__((address_space(3))) float lds_f;
        typedef __attribute__((address_space(3))) float2_t lds_f2;
        typedef __attribute__((address_space(3))) float4_t lds_f4;
        const float l = across_sum(l_run);
        if (blk == 0) *(lds_f2*)(kMergeBase + (unsigned)(wave * kRows + col) * 8) = float2_t{ref, l};
        lds_barrier();
        float2_t ml[kWaves];                                // of the wavefronts that share this one's row block, this lane's row
#pragma unroll
        for (int w = 0; w < kWaves; ++w) ml[w] = *(lds_f2*)(kMergeBase + (unsigned)((rb * cs + (w & (cs - 1))) * kRows + col) * 8);
        float mm = -INFINITY, ll = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) mm = fmaxf(mm, ml[w][0]);
        const float mz = mm == -INFINITY ? 0.f : mm;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) ll += w < cs ? ml[w][1] * __builtin_amdgcn_exp2f(ml[w][0] - mz) : 0.f;
        float weight = __builtin_amdgcn_exp2f(ref - mz);
        if (a.n_split == 1) weight *= 1.f / ll;
        if (a.n_split > 1 && slice == 0 && blk == 0 && row0 + col < rows_total) {
            const int j = row_token(row0 + col);
            const size_t out_row = ((size_t)done.n * a.m + j) * a.n_q_heads + hkv * qper + (row0 + col - j * qper);
            float* dst = a.partials + (out_row * a.n_split + done.split) * (D + kPartialHeader);
            dst[0] = mm;
            dst[1] = ll;
        }
        lds_barrier();                                      // the pairs are read: their room is the rows'
        if constexpr (HALF) {
            // (8 rows, one row block: all 128 channels of every wavefront at once; the parts of a row's probabilities, columns
            // q and q + 8, are added here)
            const int q = tid >> 6;
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) {
                float4_t v = o[cb];
#pragma unroll
                for (int e = 0; e < 4; ++e)             // (lane l + 8 mod 16 of the row)
                    v[e] += __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v[e]), 0x128, 0xf, 0xf, false));
                // (the pieces of row q change places by 4 q: the 32 lanes that write fill 512 bytes)
                if (col < 8) *(lds_f4*)(kMergeBase + (unsigned)(wave * 8 + col) * 512 + (unsigned)((4 * cb + blk) ^ (4 * col)) * 16) = v * weight;
            }
            lds_barrier();
            float2_t sum = {0.f, 0.f};
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
                sum += *(lds_f2*)(kMergeBase + (unsigned)(w * 8 + q) * 512 + (unsigned)((lane >> 1) ^ (4 * q)) * 16 + (lane & 1) * 8);
            if (q < rows_total) {
                const int j = row_token(q);
                const size_t out_row = ((size_t)done.n * a.m + j) * a.n_q_heads + hkv * qper + (q - j * qper);
                if (a.n_split == 1)
                    *reinterpret_cast<half2_t*>(a.out + out_row * D + 2 * lane) = __builtin_convertvector(sum, half2_t);
                else
                    *reinterpret_cast<float2_t*>(a.partials + (out_row * a.n_split + done.split) * (D + kPartialHeader) + kPartialHeader + 2 * lane) = sum;
            }
            if (!more) break;
            lds_barrier();
            continue;
        }
        int tid_o = tid, lane_o = lane;                     // (opaque, as above; all of it only where registers are short)
        if constexpr (C == 4) asm volatile("" : "+v"(tid_o), "+v"(lane_o));
        int q = tid_o >> 5;                                 // this thread's row and pair of channels
        if constexpr (C != 4) asm volatile("" : "+v"(q));
        const unsigned osrc = kMergeBase + (unsigned)q * kORow + (((unsigned)(tid_o & 31) >> 1) ^ (unsigned)q) * 16 + (tid_o & 1) * 8;
#pragma unroll
        for (int part = 0; part < 2; ++part) {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const float4_t v = o[4 * part + h];
                // (16-byte pieces of a row change places by the row's number: 16 rows, 16 different banks)
                *(lds_f4*)(kMergeBase + (unsigned)(wave * kRows + (lane_o & 15)) * kORow + (unsigned)((4 * h + (lane_o >> 4)) ^ (lane_o & 15)) * 16) = v * weight;
            }
            lds_barrier();
            float2_t sum = {0.f, 0.f};
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                sum += *(lds_f2*)(osrc + (unsigned)(w * kRows) * kORow);
                if (((w + 1) & (cs - 1)) != 0) continue;    // (the row block's last slice)
                const int r2 = (w >> (3 - rb_log2)) * kRows + q;
                if (r2 < rows_total) {
                    const int j = row_token(r2);
                    const size_t out_row = ((size_t)done.n * a.m + j) * a.n_q_heads + hkv * qper + (r2 - j * qper);
                    const int ch = part * 64 + 2 * (tid_o & 31);
                    if (a.n_split == 1)
                        *reinterpret_cast<half2_t*>(a.out + out_row * D + ch) = __builtin_convertvector(sum, half2_t);
                    else
                        *reinterpret_cast<float2_t*>(a.partials + (out_row * a.n_split + done.split) * (D + kPartialHeader) + kPartialHeader + ch) = sum;
                }
                sum = float2_t{0.f, 0.f};
            }
            lds_barrier();
        }
        if (!more) break;
    }
}

// At most 4 rows: lane = token, as in the decode kernel for four query heads (cq_decode_quad.hip, which says how): a token's
// scores of the four rows in the registers of its lane, by v_mfma_f32_4x4x4_16B_f16 with the queries broadcast; every
// wavefront a tile of the item by itself; probabilities relative to a running reference that moves when a score
// exceeds it by 3, as three fp16 numbers each (33 bits; twelve columns) to a [token][column] array in LDS and back transposed.
// The kernel above computes sixteen columns of softmax whatever the rows, and is bound by the vector ALU as much as by the
// LDS then: CQ-4c8b 408 instructions per tile (here 290) next to 454 clocks of LDS, 656 clocks taken, 520 here.  Measured, above
// -> here: CQ-4c8b, 32 heads, 3 tokens of 16 x 4096 50.5 -> 43.1 us, of 64 x 1000 71.7 -> 58.5; CQ-8c8b, 4 tokens of 16 x 4096 37.8 ->
// 33.8, of 64 x 1000 55.3 -> 49.9; of 4 x 30000 130 / 130 and 77 / 78.  (The same for eight rows, two fp16 numbers each and
// twice the matrix instructions, 0.94 to 1.01 times as fast as above: there the columns are no waste.)
constexpr unsigned kFewWaveBytes = 2048;                // of a wavefront: 64 tokens x 16 columns; at the end of an item four output rows
constexpr unsigned kFewPairs = kMergeBase + kWaves * kFewWaveBytes;
constexpr unsigned kFewLds = kFewPairs + kWaves * 4 * 8;
static_assert(kTileTokens * 32 == kFewWaveBytes && 4 * 128 * 4 == kFewWaveBytes, "a wavefront's room");

template <int C>
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(kWaves * 64) void chunk_few_kernel(ChunkArgs a, int per_head, int items)
{
    constexpr int D = 128, GH = D / C, K = 256, PL = GH / 16, NT = kWaves * 64, ROWS = 4, PARTS = 3;
    constexpr int TILE_BYTES = kTileTokens * GH;
    typedef __attribute__((address_space(3))) u32x4 lds_q;
    typedef __attribute__((address_space(3))) float lds_f;
    typedef __attribute__((address_space(3))) float2_t lds_f2;
    typedef __attribute__((address_space(3))) float4_t lds_f4;
    extern __shared__ float smem[];
    (void)smem;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, blk = lane >> 4;
    const int hkv = blockIdx.x % a.f.n_kv_heads;
    int item = blockIdx.x / a.f.n_kv_heads;
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    const int rows_total = a.m * qper;
    const float inv_qper = 1.f / (float)qper;
    const auto row_token = [&](int row) { return (int)(((float)row + 0.5f) * inv_qper); };     // row / qper (few rows: exact)

    // ---- both codebooks of the head on their way to LDS, ahead of the first codes, which come from further away
    u32x4 book[2][8];
    {
        const u32x4* src[2] = {reinterpret_cast<const u32x4*>(a.k_centroids + (size_t)hkv * GH * K * C),
                               reinterpret_cast<const u32x4*>(a.v_centroids + (size_t)hkv * GH * K * C)};
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll
            for (int i = 0; i < 8; ++i) book[w][i] = src[w][i * NT + tid];
    }

    // ---- this lane's places: keys, token `lane`; values, tokens 32 t + 8 blk + 4 r + col / 4, channels 4 (col % 4) .. of 16
    // (C = 8: half of group (col % 4) / 2, then every second group; C = 4: group col % 4, then every fourth)
    Unrotate unrot;
    unrot.bytes = (unsigned)(GH - lane) & 3u;
    unrot.dwords = ((unsigned)(GH - lane) & (unsigned)(GH - 1)) >> 2;
    const int vg0 = C == 8 ? (col & 3) >> 1 : (col & 3);
    const int u0 = 8 * blk + (col >> 2);
    const CodePick<GH, C == 8 ? 2 : 4> pick0(vg0, u0), pick1(vg0, u0 + 4);
    const unsigned vbase = kBookBytes + (C == 8 ? (unsigned)vg0 * 4096 + (unsigned)(col & 1) * 8 : (unsigned)vg0 * 2048);
    // (a token's 32 bytes of probabilities: halves exchanged for every second run of eight tokens, for the banks)
    const unsigned work = kMergeBase + (unsigned)wave * kFewWaveBytes;
    const unsigned prob_in = work + (unsigned)lane * 32, prob_swap = (unsigned)((lane >> 3) & 1) * 16;
    const unsigned prob_out = work + (unsigned)u0 * 32 + (((unsigned)(col & 3) * 8) ^ (unsigned)(blk & 1) * 16);

    struct Item {
        int n, split, t_n, tile0, tile1, n_tiles;
    };
    half4_t qreg[2];                                    // channels 4 (16 r + lane / 4) .. of row lane % 4
    Tile<GH, 8> krec;
    u32x4 vrec[2][2][PL];
    auto request = [&](const Item& it, int tile) {
        const size_t at = a.map.tile_index(it.n, hkv, min(tile, it.n_tiles - 1)) * TILE_BYTES;
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) krec.lo[pl] = *reinterpret_cast<const u32x4*>(a.k_codes + at + pl * 1024 + lane * 16);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int rr = 0; rr < 2; ++rr)
#pragma unroll
                for (int pl = 0; pl < PL; ++pl)
                    vrec[t][rr][pl] = *reinterpret_cast<const u32x4*>(a.v_codes + at + pl * 1024 + (32 * t + 4 * rr + u0) * 16);
    };
    auto open_item = [&](int at) {
        Item it;
        it.split = at % a.n_split;
        it.n = at / a.n_split;
        it.t_n = a.t;
        if (a.seq_lens) it.t_n = min(max(a.seq_lens[it.n], a.m), a.t);
        it.n_tiles = (it.t_n + kTileTokens - 1) / kTileTokens;
        it.tile0 = it.split * a.tiles_per_split;
        it.tile1 = min(it.tile0 + a.tiles_per_split, it.n_tiles);
        const int row = min(lane & 3, rows_total - 1), j = row_token(row);
        const uint16_t* qrow = a.q + (((size_t)it.n * a.m + j) * a.n_q_heads + hkv * qper + (row - j * qper)) * D;
#pragma unroll
        for (int i = 0; i < 2; ++i) qreg[i] = *reinterpret_cast<const half4_t*>(qrow + 64 * i + 4 * (lane >> 2));
        request(it, it.tile0 + wave);
        return it;
    };
    Item it = open_item(item);
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int i = 0; i < 8; ++i) *(lds_q*)(w * kBookBytes + (unsigned)(i * NT + tid) * 16) = book[w][i];
    lds_barrier();

#pragma unroll 1
    for (;;) {
        float4_t o[8];
#pragma unroll
        for (int cb = 0; cb < 8; ++cb) o[cb] = float4_t{0.f, 0.f, 0.f, 0.f};
        float ref[ROWS], l[ROWS];                           // (l: this lane's tokens)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            ref[r] = kNoScore;
            l[r] = 0.f;
        }
        unsigned d[GH / 4], z[2][2][2];                     // codes of the tile to come: keys in group order, values as picked
        auto unpack = [&]() {
            group_order<GH, 8>(krec, unrot, d);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                pick0(vrec[t][0], 0, z[t][0]);
                pick1(vrec[t][1], 0, z[t][1]);
            }
        };
        const int pos0 = it.t_n - a.m;                      // position of query token 0
        int tile = it.tile0 + wave;
        bool turn = wave < kWaves / 2;                      // (priorities as in cq_decode_quad.hip)
        unpack();
        request(it, tile + kWaves);
#pragma unroll 1
        for (; tile < it.tile1; tile += kWaves) {
            turn = !turn;
            if (turn) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
            // ---- scores of the lane's token
            float4_t acc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = float4_t{0.f, 0.f, 0.f, 0.f};
            {
                unsigned at[GH];
#pragma unroll
                for (int g = 0; g < GH; ++g) at[g] = entry<C>(d[g >> 2], g & 3, 0u);
                __builtin_amdgcn_sched_barrier(0);          // (addresses first: a gather right behind its own would wait for it)
                CenVec<C> kv[GH];
#pragma unroll
                for (int g = 0; g < GH; ++g) kv[g] = lds_centroid<C>(at[g] + (unsigned)g * (K * C * 2));
                __builtin_amdgcn_sched_barrier(0);
                typedef unsigned u2 __attribute__((ext_vector_type(2)));
#pragma unroll
                for (int g = 0; g < GH; ++g)
#pragma unroll
                    for (int p = 0; p < C / 4; ++p) {
                        const int i = g * (C / 4) + p;
                        acc[i & 3] = mfma_quad(qreg, __builtin_bit_cast(half4_t, u2{kv[g].w[2 * p], kv[g].w[2 * p + 1]}), acc[i & 3], i);
                    }
            }
            // ---- the values of tokens 0-31 on their way
            half8_t av[2][8];
            auto gather = [&](int t) {
                unsigned at[2][8];
#pragma unroll
                for (int rr = 0; rr < 2; ++rr)
#pragma unroll
                    for (int cb = 0; cb < 8; ++cb) at[rr][cb] = entry<C>(z[t][rr][cb >> 2], cb & 3, vbase);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int cb = 0; cb < 8; ++cb) {
                    const half4_t v0 = lds_transposed(at[0][cb] + (unsigned)cb * 8192), v1 = lds_transposed(at[1][cb] + (unsigned)cb * 8192);
                    av[t][cb] = half8_t{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            if (turn) __builtin_amdgcn_s_setprio(3);
            else __builtin_amdgcn_s_setprio(2);
            gather(0);
            // ---- softmax
            float s[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) s[r] = ((acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r])) * a.scale_log2e;
            if (tile * kTileTokens + kTileTokens - 1 > pos0) {      // (some row does not see all of this tile)
                const int tok = tile * kTileTokens + lane;
#pragma unroll
                for (int r = 0; r < ROWS; ++r) s[r] = tok <= pos0 + row_token(min(r, rows_total - 1)) ? s[r] : -INFINITY;
            }
            float over = s[0] - ref[0];
#pragma unroll
            for (int r = 1; r < ROWS; ++r) over = fmaxf(over, s[r] - ref[r]);
            if (__builtin_amdgcn_ballot_w64(over > 3.f) != 0) {
                float mine = 1.f;
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    const float top = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(fmaxf(ref[r], wave_max(s[r])))));
                    const float alpha = __builtin_amdgcn_exp2f(ref[r] - top);
                    l[r] *= alpha;
                    ref[r] = top;
                    mine = (lane & (ROWS - 1)) == r ? alpha : mine;
                }
#pragma unroll
                for (int cb = 0; cb < 8; ++cb) o[cb] *= mine;
            }
            // p 2^12 as the sum of three fp16 numbers (what is left over each time is exact)
            unsigned part[PARTS][ROWS / 2];
#pragma unroll
            for (int r = 0; r < ROWS; r += 2) {
                float2_t p;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    p[e] = __builtin_amdgcn_exp2f(s[r + e] - ref[r + e]) * 4096.f;     // (12 in the exponent would be lost in a large reference)
                    l[r + e] += p[e];
                }
#pragma unroll
                for (int k = 0; k < PARTS; ++k) {
                    const half2_t v = __builtin_convertvector(p, half2_t);
                    part[k][r >> 1] = __builtin_bit_cast(unsigned, v);
                    if (k + 1 < PARTS) p = float2_t{__builtin_fmaf((float)v.x, -1.f, p[0]), __builtin_fmaf((float)v.y, -1.f, p[1])};
                }
            }
            // (a wavefront's LDS operations keep their order; the statements keep the compiler from moving the reads, which
            // are of what other lanes wrote)
            *(lds_q*)(prob_in + prob_swap) = u32x4{part[0][0], part[0][1], part[1][0], part[1][1]};
            *(lds_q*)(prob_in + (prob_swap ^ 16u)) = u32x4{part[2][0], part[2][1], 0u, 0u};
            asm volatile("" ::: "memory");
            half8_t pb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const half4_t v0 = lds_transposed(prob_out + (unsigned)t * 1024), v1 = lds_transposed(prob_out + (unsigned)t * 1024 + 128);
                pb[t] = half8_t{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
            }
            asm volatile("" ::: "memory");
            gather(1);
            // ---- O^T += V^T P
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int cb = 0; cb < 8; ++cb) o[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[t][cb], pb[t], o[cb], 0, 0, 0);
            // the next tile's codes, and the request for the tile after it
            unpack();
            request(it, tile + 2 * kWaves);
        }

        // ---- the next item's requests go out, then the wavefronts are merged
        const Item done = it;
        item += per_head;
        const bool more = item < items;
        if (more) it = open_item(item);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const float sum = wave_sum(l[r]);
            if (lane == 0) *(lds_f2*)(kFewPairs + (unsigned)(wave * ROWS + r) * 8) = float2_t{ref[r], sum};
        }
        // (the parts of a row are columns r, r + 4, r + 8)
#pragma unroll
        for (int cb = 0; cb < 8; ++cb) {
            float4_t v = o[cb];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] += __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v[e]), 0x128, 0xf, 0xf, false));    // row_ror:8
                v[e] += __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v[e]), 0x124, 0xf, 0xf, false));    // row_ror:4
            }
            if (col < ROWS) *(lds_f4*)(work + (unsigned)(col * D + 16 * cb + 4 * blk) * 4) = v;
        }
        lds_barrier();
        static_assert(NT == ROWS * D, "one output per thread");
        const int r = tid / D, ch = tid % D;
        float2_t ml[kWaves];
        float m = kNoScore;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            ml[w] = *(lds_f2*)(kFewPairs + (unsigned)(w * ROWS + r) * 8);
            m = fmaxf(m, ml[w][0]);
        }
        float sum = 0.f, ll = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float weight = __builtin_amdgcn_exp2f(ml[w][0] - m);
            sum = __builtin_fmaf(*(lds_f*)(kMergeBase + (unsigned)(w * ROWS * D + tid) * 4), weight, sum);
            ll = __builtin_fmaf(ml[w][1], weight, ll);
        }
        if (r < rows_total) {
            const int j = row_token(r);
            const size_t out_row = ((size_t)done.n * a.m + j) * a.n_q_heads + hkv * qper + (r - j * qper);
            if (a.n_split == 1) {
                a.out[out_row * D + ch] = __builtin_bit_cast(uint16_t, (_Float16)(sum / ll));
            } else {                                    // (a row that sees no token of the split: no weight)
                float* dst = a.partials + (out_row * a.n_split + done.split) * (D + kPartialHeader);
                if (ch == 0) {
                    dst[0] = m;
                    dst[1] = ll * 0x1p-12f;
                }
                dst[kPartialHeader + ch] = sum * 0x1p-12f;
            }
        }
        if (!more) break;
        lds_barrier();                                  // the rows and pairs are read: their room is the next item's
    }
}

template <class Kernel>
cq_status launch(Kernel kernel, LdsKernelSetup& setup, unsigned lds, const ChunkArgs& a, hipStream_t stream, bool few)
{
    if (setup.ensure(reinterpret_cast<const void*>(kernel)) != hipSuccess) return CQ_ERR_HIP;
    const ChunkLdsPlan p = chunk_lds_plan(a.f, a.n_q_heads, a.m);
    const int items = a.batch * a.n_split;
    const int per_head = items < p.wgs_per_head ? items : p.wgs_per_head;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(per_head * a.f.n_kv_heads)), dim3(kWaves * 64), lds, stream, a, few ? per_head : p.rb_log2, items);
    return hipGetLastError() == hipSuccess ? CQ_OK : CQ_ERR_HIP;
}

template <int C>
cq_status launch_rows(const ChunkArgs& a, int rows, hipStream_t stream)
{
    static LdsKernelSetup setup[3];
    if (rows <= 4) return launch(chunk_few_kernel<C>, setup[0], kFewLds, a, stream, true);
    if (rows <= kRows / 2) return launch(chunk_lds_kernel<C, true>, setup[1], kLdsBytes, a, stream, false);
    return launch(chunk_lds_kernel<C, false>, setup[2], kLdsBytes, a, stream, false);
}

}  // namespace

ChunkLdsPlan chunk_lds_plan(const Derived& f, int n_q_heads, int m)
{
    ChunkLdsPlan p;
    const int blocks = (m * (n_q_heads / f.n_kv_heads) + kRows - 1) / kRows;
    p.rb_log2 = blocks <= 1 ? 0 : (blocks <= 2 ? 1 : 2);
    p.wgs_per_head = f.n_kv_heads < 256 ? 256 / f.n_kv_heads : 1;      // one workgroup per CU
    return p;
}

cq_status launch_chunk_lds(const ChunkArgs& a, hipStream_t stream)
{
    // (row / qper is formed in floating point: exact for far more rows than are served here)
    const int64_t rows = (int64_t)a.m * (a.n_q_heads / a.f.n_kv_heads);
    if (a.f.b != 8 || a.f.head_dim != 128 || rows > kChunkLdsRows) return CQ_ERR_UNSUPPORTED;
    if (a.f.c == 8) return launch_rows<8>(a, (int)rows, stream);
    if (a.f.c == 4) return launch_rows<4>(a, (int)rows, stream);
    return CQ_ERR_UNSUPPORTED;
}

}  // namespace cq
