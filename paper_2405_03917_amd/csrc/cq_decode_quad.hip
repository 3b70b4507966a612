// Decode attention with grouped queries, both codebooks of a KV head in LDS, for gfx950: the (up to) four query heads
// of a KV head that a workgroup serves share every code load, every gathered key and value and (keys cached before the
// rotary embedding) every key rotation.  The formats whose two codebooks fit: CQ-8c8b and CQ-4c8b (2 x 64 KB of the
// CU's 160 KB).
//
// A codebook belongs to the KV head and not to the sequence, so a workgroup brings both in ONCE and then walks
// (sequence, split) items of its KV head; no table is built per sequence and query head.  Within an item every
// wavefront takes every eighth 64-token tile by itself, keys, softmax and values, with no barrier in the loop:
//   scores   lane = token.  A lane reads the centroids of its token's codes (ds_read_b128 / b64); a product of four
//            heads x 4 channels with 4 channels x 4 tokens per block of four lanes (v_mfma_f32_4x4x4_16B_f16, the
//            queries broadcast from one block) leaves a token's four scores in its lane's four registers.
//            ROPE: the key is rotated by the lane's part of its position and each head's query by the tile's
//            (cq_decode_rope.hip), products of one channel each in fp32 (v_mfma_f32_4x4x1_16B_f32).
//   softmax  relative to a running reference per head that moves only when a score exceeds it by 3 (factor 8):
//            probabilities scaled by 2^12, three fp16 parts each (33 bits), twelve of sixteen columns of a
//            [token][column] array in LDS, read back transposed
//   values   O^T[channel][column] += V^T[channel][token] P[token][column], v_mfma_f32_16x16x32_f16; the transposing
//            read gathers the centroids of 4 tokens per lane group
// The wavefronts are merged through LDS at the end of an item; the partials of several splits by a kernel of its own
// (counting workgroups in and merging in the last of them, as cq_decode.hip does, took 1 to 3 us longer here).
//
// Bound, keys as stored: the LDS.  A tile costs a CU 434 (CQ-8c8b) or 476 (CQ-4c8b) clocks of it, 270 to 320 of them bank
// conflicts of the gathers: 64 random 8-byte entries take 6.2 to 7 clocks instead of 2, 16-byte ones 12 instead of 4 (other
// places of the entries, by group or code, 5.7 to 6.4).  Measured: the paged fused step of CQ-4c8b, 32 / 8 heads, 24 ragged
// rows to 6007, 44.4 us with a workgroup and tables per query head -> 30.5 here: launch 2.7, codebooks 2.8, search for the
// new token's codes 3, 22 for the 94 tiles of the longest row (LDS busy throughout), merge 1.
// ROPE: issue of vector and matrix instructions, 576 and 144 per tile, which hardly overlap: 2304 + 1280 of 3800 clocks per
// tile and SIMD.  The fused step of CQ-8c8b, 32 / 8 heads, 32 x 16384: 161.4 us with the phases one after the other in a
// workgroup (scores of a split to LDS, the value codebook in the key codebook's place) -> 112.  On the way: splits
// that one workgroup walks joined 143 -> 121; priorities 121 -> 116; nothing spilled ahead of the first requests 118 -> 112.
// Priorities: the two wavefronts of a SIMD should be in different phases, and neither may fall behind (an item ends
// with its slowest wavefront).  A wavefront's priority is high in its latency-bound half of a tile (softmax, values), and
// within both halves the wavefronts take turns from tile to tile: with none, wavefront 0 waited 26 of 130 us for the
// others of its workgroup; now 2.5.
#include <type_traits>

#include "cq_decode_split.hpp"
#include "cq_key_gather.hpp"
#include "cq_lds_gather.hpp"

namespace cq {
namespace {

constexpr int kQuadThreads = 512;
constexpr int kQuadHeads = 4;
constexpr int kQuadWaves = kQuadThreads / 64;
// LDS: key codebook, value codebook, per wavefront 2 KB (probabilities of a tile, 64 tokens x 16 columns; at the end of
// an item its four output rows), the wavefronts' (reference, sum) pairs, the new token's minima
constexpr unsigned kQuadWaveBytes = 2048;
constexpr unsigned kQuadWork = 2 * kBookBytes;
constexpr unsigned kQuadPairs = kQuadWork + kQuadWaves * kQuadWaveBytes;
constexpr unsigned kQuadKeys = kQuadPairs + kQuadWaves * kQuadHeads * 8;
// ROPE: cosines and sines of the lanes' positions for the last kTrigPairs channel pairs; those of the others stay in
// registers, which have no room for all (77 to 134 spilled)
constexpr int kTrigPairs = 24;
constexpr unsigned kQuadTrig(int gh) { return kQuadKeys + 2 * (unsigned)gh * 8; }
constexpr unsigned kQuadLds(int gh, bool rope) { return kQuadTrig(gh) + (rope ? kTrigPairs * 64 * 8 : 0); }
static_assert(kQuadLds(32, true) <= 160 * 1024, "LDS of a CU");
static_assert(kQuadHeads * 128 * 4 == kQuadWaveBytes && kTileTokens * 32 == kQuadWaveBytes, "a wavefront's room");

// minimum over 2^STEPS neighbouring lanes
template <int STEPS>
__device__ __forceinline__ unsigned long long lanes_min_u64(unsigned long long v)
{
    auto smaller = [](unsigned long long k, unsigned lo, unsigned hi) {
        const unsigned long long o = ((unsigned long long)hi << 32) | lo;
        return o < k ? o : k;
    };
    v = smaller(v, dpp_from<0xB1>((unsigned)v), dpp_from<0xB1>((unsigned)(v >> 32)));       // quad_perm [1,0,3,2]
    v = smaller(v, dpp_from<0x4E>((unsigned)v), dpp_from<0x4E>((unsigned)(v >> 32)));       // quad_perm [2,3,0,1]
    v = smaller(v, dpp_from<0x141>((unsigned)v), dpp_from<0x141>((unsigned)(v >> 32)));     // row_half_mirror
    v = smaller(v, dpp_from<0x140>((unsigned)v), dpp_from<0x140>((unsigned)(v >> 32)));     // row_mirror
    if constexpr (STEPS == 5) {
        const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(v >> 32), (unsigned)(v >> 32), false, false);
        const unsigned long long a = ((unsigned long long)hi[0] << 32) | lo[0], b = ((unsigned long long)hi[1] << 32) | lo[1];
        v = a < b ? a : b;
    }
    return v;
}

// This lane's and thread's number for what is done once per item (`turn`) at a place (SITE) of the kernel.  ROPE forms them anew:
// kept through the tiles, they and what is derived from them would be spilled, and a spilled register comes back behind
// every load under way.  (The fused step of CQ-8c8b spilled 60, and its first codes were requested when the codebooks had
// arrived: 32 / 8 heads, 8 x 4939 27.5 -> 22.2 us without, 32 x 16384 117.6 -> 112.3.)
struct Place {
    int lane, tid;
};
template <bool ROPE, int SITE>
__device__ __forceinline__ Place place(int turn, int wave)
{
    if constexpr (!ROPE) return Place{(int)threadIdx.x & 63, (int)threadIdx.x};
    unsigned zero;
    asm("v_mov_b32 %0, 0 ; %1 %2" : "=v"(zero) : "s"(turn), "n"(SITE));
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
    return Place{lane, 64 * wave + lane};
}

template <int GH, int C, bool ROPE, bool STEP, bool LAYERS>
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(kQuadThreads) void decode_quad_kernel(
    DecodeArgs a, const float2* tile_tab, const float2* lane_tab, int items, int per_head)
{
    constexpr int NT = kQuadThreads, NW = kQuadWaves, QH = kQuadHeads, D = 128, K = 256, PL = GH / 16, HALF = GH / 2;
    constexpr int TILE_BYTES = kTileTokens * GH;
    static_assert(GH * C == D, "head_dim 128");
    typedef __attribute__((address_space(3))) u32x4 lds_q;
    typedef __attribute__((address_space(3))) float lds_f;
    typedef __attribute__((address_space(3))) float2_t lds_f2;
    typedef __attribute__((address_space(3))) float4_t lds_f4;
    extern __shared__ float smem[];
    unsigned long long* keys = reinterpret_cast<unsigned long long*>(smem + kQuadKeys / 4);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, blk = lane >> 4;

    // ---- workgroup -> (layer, KV head, quad of its query heads, first item); neighbouring workgroups serve different KV
    // heads, so that (a multiple of 8 of them) all workgroups of a KV head sit on one XCD and share its L2
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    const int quads = (qper + QH - 1) / QH;
    const int nh = a.f.n_kv_heads * quads;
    int r = blockIdx.x;
    int layer = 0;
    if constexpr (LAYERS) {
        layer = r / (nh * per_head);
        r -= layer * (nh * per_head);
    }
    const int hkv = (r % nh) % a.f.n_kv_heads, quad = (r % nh) / a.f.n_kv_heads;
    int item = r / nh;
    const int hq0 = hkv * qper + quad * QH;
    const int heads = min(QH, qper - quad * QH);

    const uint16_t* q_ptr = a.q;
    const uint16_t* xk_ptr = a.xk_new;
    const uint16_t* xv_ptr = a.xv_new;
    const uint8_t* k_codes = a.k_codes;
    const uint8_t* v_codes = a.v_codes;
    const uint16_t* k_centroids = a.k_centroids;
    const uint16_t* v_centroids = a.v_centroids;
    uint16_t* out_ptr = a.out;
    if constexpr (LAYERS) {
        const LayerPtrsGlobal lp = reinterpret_cast<const LayerPtrsGlobal*>(a.layers)[layer];
        q_ptr = (const uint16_t*)lp.q;
        xk_ptr = (const uint16_t*)lp.xk_new;
        xv_ptr = (const uint16_t*)lp.xv_new;
        k_codes = (const uint8_t*)lp.k_codes;
        v_codes = (const uint8_t*)lp.v_codes;
        k_centroids = (const uint16_t*)lp.k_centroids;
        v_centroids = (const uint16_t*)lp.v_centroids;
        out_ptr = (uint16_t*)lp.out;
    }

    // ---- both codebooks to LDS as they are ([group][code] entries)
    u32x4 book[2][8];
    {
        const u32x4* src[2] = {reinterpret_cast<const u32x4*>(k_centroids + (size_t)hkv * GH * K * C),
                               reinterpret_cast<const u32x4*>(v_centroids + (size_t)hkv * GH * K * C)};
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll
            for (int i = 0; i < 8; ++i) book[w][i] = src[w][i * NT + tid];
    }

    // ---- this lane's places.  Keys: token `lane` of a tile.  Values: tokens 32 t + 8 blk + 4 r + col / 4 for t, r = 0, 1;
    // channels 4 (col % 4) .. of 16 (C = 8: half of group (col % 4) / 2, then every second group; C = 4: group col % 4,
    // then every fourth)
    Unrotate unrot;
    unrot.bytes = (unsigned)(GH - lane) & 3u;
    unrot.dwords = ((unsigned)(GH - lane) & (unsigned)(GH - 1)) >> 2;
    const int vg0 = C == 8 ? (col & 3) >> 1 : (col & 3);
    const int u0 = 8 * blk + (col >> 2);
    const CodePick<GH, C == 8 ? 2 : 4> pick0(vg0, u0), pick1(vg0, u0 + 4);
    const unsigned vbase = kBookBytes + (C == 8 ? (unsigned)vg0 * 4096 + (unsigned)(col & 1) * 8 : (unsigned)vg0 * 2048);
    // probabilities: token's row of 32 bytes, its halves exchanged for every second run of eight tokens (eight lanes'
    // first halves and the next eight's second halves then lie in different banks)
    const unsigned work = kQuadWork + (unsigned)wave * kQuadWaveBytes;
    const unsigned prob_in = work + (unsigned)lane * 32, prob_swap = (unsigned)((lane >> 3) & 1) * 16;
    const unsigned prob_out = work + (unsigned)u0 * 32 + (((unsigned)(col & 3) * 8) ^ (unsigned)(blk & 1) * 16);

    // ---- an item: its places, queries, the new token's rows, its first tile's records
    struct Item {
        int n, split, t_n, tile0, tile1, n_tiles;
    };
    half4_t qreg[2];                                    // channels 4 (16 r + lane / 4) .. of head lane % 4
    uint16_t qrope[2][4];                               // ROPE: both channels of pairs lane / 4 + 16 m of head lane % 4
    Tile<GH, 8> krec, vtok;                             // vtok, cs_next: ROPE
    u32x4 vrec[2][2][PL];
    float2 cs_next[4];
    // STEP: the new token's rows: the group that this thread searches; ROPE, for want of registers: a dword of the wavefront's
    // 16 channels (of the groups that it searches), keys in lanes 0-7 of 16, values in lanes 8-15
    unsigned xrow[2][ROPE ? 1 : C / 2];
    auto request = [&](const Item& it, int tile) {
        const size_t at = a.map.tile_index(it.n, hkv, min(tile, it.n_tiles - 1)) * TILE_BYTES;
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) krec.lo[pl] = *reinterpret_cast<const u32x4*>(k_codes + at + pl * 1024 + lane * 16);
        if constexpr (!ROPE) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int rr = 0; rr < 2; ++rr)
#pragma unroll
                    for (int pl = 0; pl < PL; ++pl)
                        vrec[t][rr][pl] = *reinterpret_cast<const u32x4*>(v_codes + at + pl * 1024 + (32 * t + 4 * rr + u0) * 16);
        } else {
#pragma unroll
            for (int pl = 0; pl < PL; ++pl) vtok.lo[pl] = *reinterpret_cast<const u32x4*>(v_codes + at + pl * 1024 + lane * 16);
            const float2* row = tile_tab + (size_t)min(tile, it.n_tiles - 1) * kPairs + (lane >> 2);
#pragma unroll
            for (int m = 0; m < 4; ++m) cs_next[m] = row[16 * m];
        }
    };
    auto open_item = [&](int at) {
        const auto [lane, tid] = place<ROPE, 0>(at, wave);
        Item it;
        it.split = at % a.n_split;
        it.n = at / a.n_split;
        it.t_n = a.t;
        if (a.seq_lens) it.t_n = min(max(a.seq_lens[it.n] - a.seq_len_shift, a.seq_len_floor), a.t);
        it.n_tiles = (it.t_n + kTileTokens - 1) / kTileTokens;
        it.tile0 = it.split * a.tiles_per_split;
        it.tile1 = min(it.tile0 + a.tiles_per_split, it.n_tiles);
        const uint16_t* qrow = q_ptr + (size_t)it.n * a.q_batch_stride + (size_t)(hq0 + min(lane & 3, heads - 1)) * D;
        if constexpr (ROPE) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                qrope[0][m] = qrow[16 * m + (lane >> 2)];
                qrope[1][m] = qrow[16 * m + (lane >> 2) + kPairs];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) qreg[i] = *reinterpret_cast<const half4_t*>(qrow + 64 * i + 4 * (lane >> 2));
        }
        if constexpr (STEP) {
            const size_t at_head = (size_t)it.n * a.x_new_stride + (size_t)hkv * D;
            if constexpr (ROPE) {
                const uint16_t* row = (lane & 8) ? xv_ptr : xk_ptr;
                xrow[0][0] = *reinterpret_cast<const unsigned*>(row + at_head + 16 * wave + 2 * (lane & 7));
            } else {
                const int g = tid / (NT / GH);
#pragma unroll
                for (int i = 0; i < C / 2; ++i) {
                    xrow[0][i] = reinterpret_cast<const unsigned*>(xk_ptr + at_head + g * C)[i];
                    xrow[1][i] = reinterpret_cast<const unsigned*>(xv_ptr + at_head + g * C)[i];
                }
            }
        }
        request(it, it.tile0 + wave);
        return it;
    };
    Item it = open_item(item);

    constexpr int kHeld = kPairs - kTrigPairs;
    float cu[ROPE ? kHeld : 1], su[ROPE ? kHeld : 1];
    if constexpr (ROPE) {
#pragma unroll
        for (int i = 0; i < kHeld; ++i) {
            const float2 t = lane_tab[i * 64 + lane];
            cu[i] = t.x;
            su[i] = t.y;
        }
        static_assert(kTrigPairs * 64 % NT == 0, "whole rounds");
        float2 t[kTrigPairs * 64 / NT];
#pragma unroll
        for (int i = 0; i < kTrigPairs * 64 / NT; ++i) t[i] = lane_tab[kHeld * 64 + i * NT + tid];
#pragma unroll
        for (int i = 0; i < kTrigPairs * 64 / NT; ++i) *(lds_f2*)(kQuadTrig(GH) + (unsigned)(i * NT + tid) * 8) = float2_t{t[i].x, t[i].y};
    }
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int i = 0; i < 8; ++i) *(lds_q*)(w * kBookBytes + (unsigned)(i * NT + tid) * 16) = book[w][i];
    lds_barrier();

#pragma unroll 1
    for (;;) {
        // ---- fused step: the new token's codes, if its position lies in this item (cq_encode's arithmetic and tie rule)
        const int pos_new = it.t_n - 1;
        const int tile_new = pos_new / kTileTokens, u_new = pos_new % kTileTokens;
        const bool has_new = STEP && tile_new >= it.tile0 && tile_new < it.tile1;
        if (has_new) {
            constexpr int TPG = NT / GH;
            const auto [lane, tid] = place<ROPE, 1>(item, wave);
            const int g = tid / TPG;
            // (TPG neighbouring lanes search a group, each every TPG-th centroid in ascending order)
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                float x[C];
#pragma unroll
                for (int i = 0; i < C / 2; ++i) {
                    unsigned word;
                    if constexpr (ROPE) word = (unsigned)__builtin_amdgcn_ds_bpermute((8 * w + lane / TPG * (C / 2) + i) * 4, (int)xrow[0][0]);
                    else word = xrow[w][i];
                    const half2_t h = __builtin_bit_cast(half2_t, word);
                    x[2 * i] = (float)h.x;
                    x[2 * i + 1] = (float)h.y;
                }
                CenVec<C> cen[K / TPG];
#pragma unroll
                for (int k = 0; k < K / TPG; ++k) cen[k] = lds_centroid<C>(w * kBookBytes + (unsigned)(g * K + tid % TPG + k * TPG) * (C * 2));
                Nearest near;
#pragma unroll
                for (int k = 0; k < K / TPG; ++k) near.offer(centroid_distance<C>(x, cen[k].w), tid % TPG + k * TPG);
                const unsigned long long key = lanes_min_u64<TPG == 32 ? 5 : 4>(near.key());
                if (tid % TPG == 0) keys[w * GH + g] = key;
            }
            lds_barrier();
            if (quad == 0) {
                const size_t at = a.map.tile_index(it.n, hkv, tile_new) * TILE_BYTES;
                store_new_codes<GH, 8>(const_cast<uint8_t*>(k_codes) + at, keys, u_new, tid);
                store_new_codes<GH, 8>(const_cast<uint8_t*>(v_codes) + at, keys + GH, u_new, tid);
            }
        }

        unsigned qpair[4];                                  // ROPE: both channels in a register (here, where the codes are long under way)
        if constexpr (ROPE) {
#pragma unroll
            for (int m = 0; m < 4; ++m) qpair[m] = qrope[0][m] | (unsigned)qrope[1][m] << 16;
        }
        float4_t o[8];
#pragma unroll
        for (int cb = 0; cb < 8; ++cb) o[cb] = float4_t{0.f, 0.f, 0.f, 0.f};
        float ref[QH], l[QH];                               // per head; l: this lane's tokens
#pragma unroll
        for (int h = 0; h < QH; ++h) {
            ref[h] = kNoScore;
            l[h] = 0.f;
        }
        unsigned d[GH / 4], z[2][2][2];                     // codes of the tile to come: keys in group order, values as picked
        float qa[4], qb[4];                                 // ROPE: the queries rotated to the tile's base position
        auto unpack = [&](int tile) {
            if (has_new && tile == tile_new) {
                const int lane = place<ROPE, 2>(tile, wave).lane;
                NewTokenCodes<GH, 8> c;
                c.build(keys, u_new, lane);
                c.patch(krec, u_new, lane);
                c.build(keys + GH, u_new, lane);
                if constexpr (ROPE) {
                    c.patch(vtok, u_new, lane);
                } else {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int rr = 0; rr < 2; ++rr) {
                            const bool mine = 32 * t + 4 * rr + u0 == u_new;
#pragma unroll
                            for (int pl = 0; pl < PL; ++pl)
#pragma unroll
                                for (int i = 0; i < 4; ++i) vrec[t][rr][pl][i] = mine ? c.lo[4 * pl + i] : vrec[t][rr][pl][i];
                        }
                }
            }
            group_order<GH, 8>(krec, unrot, d);
            if constexpr (ROPE) {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const float2 t = cs_next[m];
                    const half2_t q = __builtin_bit_cast(half2_t, qpair[m]);
                    qa[m] = __builtin_fmaf((float)q.x, t.x, (float)q.y * t.y);
                    qb[m] = __builtin_fmaf((float)q.y, t.x, -((float)q.x * t.y));
                }
            } else {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    pick0(vrec[t][0], 0, z[t][0]);
                    pick1(vrec[t][1], 0, z[t][1]);
                }
            }
        };
        int tile = it.tile0 + wave;
        bool turn = wave < NW / 2;
        if constexpr (!ROPE) {
            unpack(tile);
            request(it, tile + NW);
        }
#pragma unroll 1
        for (; tile < it.tile1; tile += NW) {
            turn = !turn;
            if (turn) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
            Tile<GH, 8> vcur;
            if constexpr (ROPE) {
                unpack(tile);
                vcur = vtok;
            }
            // ---- scores of the lane's token
            float4_t acc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = float4_t{0.f, 0.f, 0.f, 0.f};
            if constexpr (ROPE) {
                // (as in decode_rope_gqa_kernel, whose comments say why the statements stand in this order)
                constexpr int kBatch = 8, GPB = kBatch / C;
                auto centroids = [&](int bi, CenVec<C> (&ka)[GPB], CenVec<C> (&kb)[GPB], float after) {
#pragma unroll
                    for (int gg = 0; gg < GPB; ++gg) {
                        const int g = bi * GPB + gg;
                        unsigned c_first = (d[g >> 2] >> (8 * (g & 3))) & 0xffu;
                        unsigned c_second = (d[(g + HALF) >> 2] >> (8 * ((g + HALF) & 3))) & 0xffu;
                        asm volatile("" : "+v"(c_first), "+v"(c_second) : "v"(after));
                        ka[gg] = lds_centroid<C>(c_first * (C * 2) + (unsigned)(g * K * C * 2));
                        kb[gg] = lds_centroid<C>(c_second * (C * 2) + (unsigned)((g + HALF) * K * C * 2));
                    }
                };
                static_assert(kHeld % kBatch == 0, "a batch's cosines and sines in one place");
                float2_t trig[kBatch];
                auto trig_of = [&](int bi, float2_t (&v)[kBatch]) {
#pragma unroll
                    for (int e = 0; e < kBatch; ++e) v[e] = *(lds_f2*)(kQuadTrig(GH) + (unsigned)((bi * kBatch - kHeld + e) * 64 + lane) * 8);
                };
                CenVec<C> ka[GPB], kb[GPB];
                centroids(0, ka, kb, 0.f);
#pragma unroll
                for (int bi = 0; bi < kPairs / kBatch; ++bi) {
                    CenVec<C> ka_n[GPB], kb_n[GPB];
                    float t1[kBatch], t2[kBatch], x[kBatch], y[kBatch];
                    const auto cosine = [&](int e) { return bi * kBatch < kHeld ? cu[bi * kBatch < kHeld ? bi * kBatch + e : 0] : trig[e][0]; };
                    const auto sine = [&](int e) { return bi * kBatch < kHeld ? su[bi * kBatch < kHeld ? bi * kBatch + e : 0] : trig[e][1]; };
#pragma unroll
                    for (int e = 0; e < kBatch; ++e) t1[e] = mixv_mul((e % C) & 1, kb[e / C].w[(e % C) >> 1], sine(e));
                    if (bi + 1 < kPairs / kBatch) centroids(bi + 1, ka_n, kb_n, t1[0]);
                    if (bi == 3) request(it, tile + NW);
#pragma unroll
                    for (int e = 0; e < kBatch; ++e) t2[e] = mixv_mul((e % C) & 1, ka[e / C].w[(e % C) >> 1], sine(e));
#pragma unroll
                    for (int e = 0; e < kBatch; ++e) x[e] = mixv_fma<true>((e % C) & 1, ka[e / C].w[(e % C) >> 1], cosine(e), t1[e]);
#pragma unroll
                    for (int e = 0; e < kBatch; ++e) y[e] = mixv_fma<false>((e % C) & 1, kb[e / C].w[(e % C) >> 1], cosine(e), t2[e]);
                    if (bi + 1 < kPairs / kBatch && (bi + 1) * kBatch >= kHeld) trig_of(bi + 1, trig);
                    static_assert(kBatch == 8, "operands of the statement below");
                    asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]),
                                      "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3]), "+v"(y[4]), "+v"(y[5]), "+v"(y[6]), "+v"(y[7]));
#pragma unroll
                    for (int e = 0; e < kBatch; ++e) {
                        const int i = bi * kBatch + e;              // pair i: register i / 16 of the block of lanes i % 16
                        acc[2 * (e & 1)] = mfma_pair(qa, x[e], acc[2 * (e & 1)], i);
                        acc[2 * (e & 1) + 1] = mfma_pair(qb, y[e], acc[2 * (e & 1) + 1], i);
                    }
                    asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));
                    if (bi + 1 < kPairs / kBatch) {
#pragma unroll
                        for (int gg = 0; gg < GPB; ++gg) { ka[gg] = ka_n[gg]; kb[gg] = kb_n[gg]; }
                    }
                }
            } else {
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
            if constexpr (ROPE) {
                // (the value codes change from their token's lane to the lanes that gather, through this wavefront's room)
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) *(lds_q*)(work + (unsigned)(pl * 1024 + lane * 16)) = vcur.lo[pl];
                asm volatile("" ::: "memory");
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    u32x4 rec[2][PL];
#pragma unroll
                    for (int rr = 0; rr < 2; ++rr)
#pragma unroll
                        for (int pl = 0; pl < PL; ++pl) rec[rr][pl] = *(lds_q*)(work + (unsigned)(pl * 1024 + (32 * t + 4 * rr + u0) * 16));
                    pick0(rec[0], 0, z[t][0]);
                    pick1(rec[1], 0, z[t][1]);
                }
                asm volatile("" ::: "memory");
            }
            gather(0);
            // ---- softmax
            float s[QH];
#pragma unroll
            for (int h = 0; h < QH; ++h) {
                s[h] = (acc[0][h] + acc[1][h]) + (acc[2][h] + acc[3][h]);
                s[h] *= a.scale_log2e;
            }
            if (tile == it.n_tiles - 1) {
                const bool live = tile * kTileTokens + lane < it.t_n;
#pragma unroll
                for (int h = 0; h < QH; ++h) s[h] = live ? s[h] : -INFINITY;
            }
            const float over = fmaxf(fmaxf(s[0] - ref[0], s[1] - ref[1]), fmaxf(s[2] - ref[2], s[3] - ref[3]));
            if (__builtin_amdgcn_ballot_w64(over > 3.f) != 0) {
                float alpha[QH];
#pragma unroll
                for (int h = 0; h < QH; ++h) {
                    const float top = fmaxf(ref[h], wave_max(s[h]));
                    alpha[h] = __builtin_amdgcn_exp2f(ref[h] - top);
                    l[h] *= alpha[h];
                    ref[h] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(top)));
                }
                const float mine = (lane & 2) ? ((lane & 1) ? alpha[3] : alpha[2]) : ((lane & 1) ? alpha[1] : alpha[0]);
#pragma unroll
                for (int cb = 0; cb < 8; ++cb) o[cb] *= mine;
            }
            // p 2^12 as the sum of three fp16 numbers (towards zero: what is left over is exact)
            unsigned part[3][2];
#pragma unroll
            for (int h = 0; h < QH; h += 2) {
                float p[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    p[e] = __builtin_amdgcn_exp2f(s[h + e] - ref[h + e]) * 4096.f;     // (12 in the exponent would be lost in a large reference)
                    l[h + e] += p[e];
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const half2_t v = __builtin_bit_cast(half2_t, __builtin_amdgcn_cvt_pkrtz(p[0], p[1]));
                    part[k][h >> 1] = __builtin_bit_cast(unsigned, v);
                    if (k < 2) {
                        p[0] = __builtin_fmaf((float)v.x, -1.f, p[0]);
                        p[1] = __builtin_fmaf((float)v.y, -1.f, p[1]);
                    }
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
            if constexpr (!ROPE) gather(1);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if constexpr (ROPE) {
                    if (t == 1) gather(1);
                }
#pragma unroll
                for (int cb = 0; cb < 8; ++cb) o[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[t][cb], pb[t], o[cb], 0, 0, 0);
            }
            // the next tile's codes, and the request for the tile after it
            if constexpr (!ROPE) {
                unpack(tile + NW);
                request(it, tile + 2 * NW);
            }
        }

        // ---- the next item's requests go out, then the wavefronts are merged
        const Item done = it;
        item += per_head;
        const bool more = item < items;
        if (more) it = open_item(item);
        const auto [lane, tid] = place<ROPE, 3>(item, wave);
        const int col = lane & 15, blk = lane >> 4;
#pragma unroll
        for (int h = 0; h < QH; ++h) {
            const float sum = wave_sum(l[h]);
            if (lane == 0) *(lds_f2*)(kQuadPairs + (unsigned)(wave * QH + h) * 8) = float2_t{ref[h], sum};
        }
        // (the parts of a head are columns h, h + 4, h + 8)
#pragma unroll
        for (int cb = 0; cb < 8; ++cb) {
            float4_t v = o[cb];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] += __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v[e]), 0x128, 0xf, 0xf, false));    // row_ror:8
                v[e] += __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v[e]), 0x124, 0xf, 0xf, false));    // row_ror:4
            }
            if (col < QH) *(lds_f4*)(work + (unsigned)(col * D + 16 * cb + 4 * blk) * 4) = v;
        }
        lds_barrier();
        static_assert(NT == QH * D, "one output per thread");
        const int h = tid / D, ch = tid % D;
        float2_t ml[NW];
        float m = kNoScore;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            ml[w] = *(lds_f2*)(kQuadPairs + (unsigned)(w * QH + h) * 8);
            m = fmaxf(m, ml[w][0]);
        }
        float sum = 0.f, ll = 0.f;                          // (a split beyond its sequence's end: m = kNoScore, both 0)
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float weight = __builtin_amdgcn_exp2f(ml[w][0] - m);
            sum = __builtin_fmaf(*(lds_f*)(kQuadWork + (unsigned)(w * QH * D + tid) * 4), weight, sum);
            ll = __builtin_fmaf(ml[w][1], weight, ll);
        }
        if (a.n_split == 1) {
            if (h < heads) out_ptr[(size_t)done.n * a.out_batch_stride + (size_t)(hq0 + h) * D + ch] = __builtin_bit_cast(uint16_t, (_Float16)(sum / ll));
        } else {
            const size_t row = ((size_t)layer * a.batch + done.n) * a.n_q_heads + hq0 + min(h, heads - 1);
            float* dst = a.partials + (row * a.n_split + done.split) * (D + kPartialHeader);
            if (h < heads) {
                if (ch == 0) {
                    dst[0] = m;
                    dst[1] = ll * 0x1p-12f;
                }
                dst[kPartialHeader + ch] = sum * 0x1p-12f;
            }
        }
        if (!more) break;
        lds_barrier();                                      // the rows and pairs are read: their room is the next item's
    }
}

// Neighbouring splits of a call join where that fills the CUs as well: a workgroup walks its items one after the other,
// and every item costs the merge of its wavefronts (about kItemTiles tiles).  Never more partials than the call's split
// has, and decided by sizes alone.  (By ceil(n_split / n), the splits to an item, of which there are about 2 sqrt(n_split): with all n
// a call over 131072 tokens in splits of 64 took 11 us on the host.)
constexpr int kItemTiles = 6;
DecodeArgs joined_splits(const DecodeArgs& a)
{
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    const int nh = a.f.n_kv_heads * ((qper + kQuadHeads - 1) / kQuadHeads), resident = nh < 256 ? 256 / nh : 1;
    const int n_tiles = (a.t + kTileTokens - 1) / kTileTokens;
    DecodeArgs best = a;
    int64_t best_cost = -1;
    for (int n = a.n_split; n >= 1;) {
        const int joined = (a.n_split + n - 1) / n, tiles = joined * a.tiles_per_split, split = (n_tiles + tiles - 1) / tiles;
        n = (a.n_split + joined - 1) / joined - 1;
        const int64_t rounds = ((int64_t)a.batch * split + resident - 1) / resident, cost = rounds * (tiles + kItemTiles);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best.tiles_per_split = tiles;
            best.n_split = split;
        }
    }
    return best;
}

template <int GH, int C, bool ROPE, bool STEP, bool LAYERS>
cq_status launch_variant(const DecodeArgs& a, const float2* tile_tab, const float2* lane_tab, hipStream_t stream)
{
    auto kernel = decode_quad_kernel<GH, C, ROPE, STEP, LAYERS>;
    static LdsKernelSetup setup;
    if (setup.ensure(reinterpret_cast<const void*>(kernel)) != hipSuccess) return CQ_ERR_HIP;
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    const int nh = a.f.n_kv_heads * ((qper + kQuadHeads - 1) / kQuadHeads);
    const int items = a.batch * a.n_split;
    const int resident = nh < 256 ? 256 / nh : 1;           // one workgroup per CU
    const int per_head = items < resident ? items : resident;
    const unsigned grid = (unsigned)(per_head * nh) * (unsigned)(LAYERS ? a.n_layers : 1);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kQuadThreads), kQuadLds(GH, ROPE), stream, a, tile_tab, lane_tab, items, per_head);
    return hipGetLastError() == hipSuccess ? CQ_OK : CQ_ERR_HIP;
}

template <bool ROPE, bool STEP, bool LAYERS>
cq_status launch_format(const DecodeArgs& a, const float2* tile_tab, const float2* lane_tab, hipStream_t stream)
{
    if (a.f.b != 8 || a.f.head_dim != 128) return CQ_ERR_UNSUPPORTED;
    if (a.f.c == 8) return launch_variant<16, 8, ROPE, STEP, LAYERS>(a, tile_tab, lane_tab, stream);
    if (a.f.c == 4) return launch_variant<32, 4, ROPE, STEP, LAYERS>(a, tile_tab, lane_tab, stream);
    return CQ_ERR_UNSUPPORTED;
}

}  // namespace

// Whether a call over keys as stored goes here rather than to the kernels with tables and bins (cq_decode.hip, cq_decode_pair.hip):
// query heads in fours, enough items for the CUs (one workgroup each, 256), and, of CQ-8c8b, splits that are short or
// fill their rounds; 32 / 8 heads, tables -> here, us per cq_decode_attention call:
//   CQ-4c8b  18 x 64 11.6 -> 7.0, 64 x 64 31.4 -> 9.7, 64 x 300 32.6 -> 11.9, 18 x 1100 17.1 -> 10.5, 64 x 1100 41.3 -> 18.6, 20 x 2000 20.9 -> 13.4,
//            12 x 8000 (two splits) 31.4 -> 22.9, 34 x 4200 49.0 -> 38.1, 48 x 16000 131 -> 116, 64 x 16000 189 -> 131; with 128 items (16
//            sequences, which fill the CUs in pairs) 300 9.1 -> 7.7, 2000 13.2 -> 13.4, 4200 18.0 -> 20.7, 16000 46.9 -> 58.7
//   CQ-8c8b  18 x 64 10.5 -> 7.1, 64 x 64 31.3 -> 8.7, 64 x 300 31.8 -> 10.9, 18 x 1100 13.0 -> 10.1, 64 x 1100 36.0 -> 17.1, 20 x 4200 22.2 -> 19.3,
//            28 x 4200 27.4 -> 19.5, 64 x 16000 123 -> 105; 128 items: 300 9.0 -> 7.2, 2000 10.9 -> 12.1
// (the fused step, with its search here, alike: 18 x 64 17.4 -> 9.6 and 15.4 -> 8.8, 34 x 2000 39.6 -> 27.9 and 29.8 -> 25.4).
// A tile of CQ-8c8b costs 434 clocks of the LDS here and 258 with tables, so long splits, as they are walked here (joined), have
// to fill their rounds: of 250 tiles 18 / 20 / 24 x 16000 50.7 / 51.7 / 51.7 -> 53.6 / 53.3 / 53.1, 28 x 16000 61.8 -> 54.1; of 125 tiles 18 x
// 8000 30.3 -> 30.1, 12 x 16000 33.0 -> 33.0; in two rounds 34 x 8000 46.3 -> 56.7, 34 x 4200 33.6 -> 34.7, 34 x 2000 21.8 -> 20.8.  One of
// CQ-4c8b costs 476 and 515.
bool decode_takes_quads(const DecodeArgs& a, DecodeArgs* joined)
{
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    if (a.f.b != 8 || a.f.c < 4 || a.f.head_dim != 128 || qper % kQuadHeads != 0) return false;
    const int64_t items_per_split = (int64_t)a.batch * (a.n_q_heads / kQuadHeads);
    if (items_per_split * a.n_split < 140) return false;
    const DecodeArgs j = joined_splits(a);
    const int64_t items = items_per_split * j.n_split, rounds = (items + 255) / 256;
    if (items < 140) return false;
    *joined = j;
    if (a.f.c == 4) return true;
    return items * 100 >= rounds * 256 * 78 || j.tiles_per_split <= (rounds == 1 ? 128 : 64);
}

cq_status launch_decode_quad(const DecodeArgs& a, hipStream_t stream)
{
    const cq_status st = a.layers   ? launch_format<false, true, true>(a, nullptr, nullptr, stream)
                         : a.xk_new ? launch_format<false, true, false>(a, nullptr, nullptr, stream)
                                    : launch_format<false, false, false>(a, nullptr, nullptr, stream);
    if (st != CQ_OK || a.n_split == 1) return st;
    return launch_decode_merge(a, stream);
}

cq_status launch_decode_quad_rope(const DecodeArgs& a_in, const float2* tile_tab, const float2* lane_tab, hipStream_t stream)
{
    // (every call of grouped queries comes here, and a given split fixes its bits in any batch: joining, which follows the
    // batch, is for the library's own split)
    const DecodeArgs a = a_in.split_given ? a_in : joined_splits(a_in);
    const cq_status st = a.xk_new ? launch_format<true, true, false>(a, tile_tab, lane_tab, stream) : launch_format<true, false, false>(a, tile_tab, lane_tab, stream);
    if (st != CQ_OK || a.n_split == 1) return st;
    return launch_decode_merge(a, stream);
}

}  // namespace cq
