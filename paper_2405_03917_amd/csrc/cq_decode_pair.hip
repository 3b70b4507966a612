// Decode attention straight from packed CQ codes for grouped queries: a workgroup of 16 wavefronts serves TWO
// query heads of a KV head (cq_decode.hip: one, and what the kernels have in common), for gfx950.
//
// What bounds grouped queries is not the code streams, which further heads of a KV head find in L2, but the LDS: a
// gather and an add per group, token and head.  The LDS reads 64 bits per lane in the time of 32 (measured, clocks
// per wavefront and CU without bank conflicts: ds_read_b32 and ds_read_b64 2.05, ds_read_b128 4.1, ds_add_u32 4.0,
// ds_add_u64 6.0), so a cell of the score table and of the bins is a pair of words here, one per head: 8.1 clocks
// for a gather and an add of both heads against 12.2, and the codes, their addresses, the codebooks and the new
// token's search are shared.  (A group of four heads would take ds_read_b128 and two ds_add_u64: as many LDS clocks per head.)
// Table and bins of CQ-8c8b and CQ-4c8b are 64 KB each (SEPARATE), those of CQ-2c8b and CQ-8c10b share 128 KB
// (SHARED): one workgroup has the CU, and nothing overlaps its table build and epilogue.
//
// Measured (32 / 8 heads; one head per workgroup -> two, both with the present kernels on one card): CQ-8c10b, batch 32 x 16384
// 103.6 -> 77.6 us (74 to 78 on other cards), its step 132.8 -> 92.4, batch 16 x 300 16.3 -> 12.2; CQ-2c8b, batch 16 x 4096
// 37.2 -> 29.5; CQ-4c8b, 32 x 16384 115.5 -> 94.0, 16 x 4096 20.3 -> 17.1; CQ-8c8b, 32 x 16384 66.2 -> 62.9.  The walk's key half is bound by the vector ALU (about 220 clocks per tile and SIMD
// against 33 of LDS per CU), its value half by the LDS (96 per CU against 170 of vector ALU per SIMD), and all wavefronts are in
// the same half.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "cq_decode_split.hpp"

namespace cq {
namespace {

constexpr int H = 2;                                    // query heads of a workgroup
constexpr int kPairThreads = kDecodeThreads * H;

// ---- layout of the workgroup's LDS
template <int GH, int B>
struct Lay {
    static constexpr int K = 1 << B;
    static constexpr int NW = kDecodeWaves * H;                     // wavefronts
    static constexpr bool SEPARATE = B == 8 && GH <= 32;            // table and bins side by side (else one after the other)
    static constexpr int R = (GH == 16 && B == 8) ? 2 : 1;          // replicas per group
    static constexpr unsigned TAB_BYTES = 131072;                   // table and bins
    static constexpr unsigned BIN_BYTES = SEPARATE ? 65536 : 0;     // the bins' cells, this far behind the table's
    static constexpr int ROW_BYTES = SEPARATE ? 256 : 512;
    static constexpr int TILE_BYTES = kTileTokens * GH * B / 8;
    static constexpr int SLOTS = TAB_BYTES / 4;                     // [2][H][2][NW] floats
    static constexpr int SUMS = SLOTS + 4 * H * NW;                 // [H][NW] unsigned
    static constexpr int SCR = SUMS + H * NW;                       // 64 + H * NW * head_dim floats
    static constexpr int KEYS(int head_dim) { return SCR + 64 + H * NW * head_dim; }   // fused step only
    // fused step: the keys, the new token's fixed-point weights, its record of key codes in cache order
    static constexpr int FLOATS(int head_dim, bool step) { return KEYS(head_dim) + (step ? NewTokenWords<GH, B>::END : 0); }
    // Byte address of the cell of code value j in column `col`.  b = 8: row j.  b = 10: row = the low 8 bits,
    // and the two high bits pick one of four 16-cell quarters of the row.
    __device__ __forceinline__ static constexpr unsigned cell(int j, int col)
    {
        return B == 8 ? (unsigned)(j * ROW_BYTES + col * 8) : (unsigned)((j & 255) * ROW_BYTES + (j >> 8) * 128 + col * 8);
    }
};

// Per-lane column constants for the Gh slots of a token, four byte offsets per register: of 8-byte columns
// (SEPARATE), or of 4-byte columns, doubled together with the code (SHARED: rows of 512 bytes).
template <int GH, int B>
struct Cols {
    unsigned v[GH / 4];
    __device__ __forceinline__ void init(int lane)
    {
#pragma unroll
        for (int i = 0; i < GH / 4; ++i) {
            unsigned x = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int g = (lane + 4 * i + k) & (GH - 1);
                const int column = Lay<GH, B>::R == 2 ? 2 * g + ((lane >> 4) & 1) : g;   // lanes l and l + 16 differ, l and l + 32 share
                x |= (unsigned)((Lay<GH, B>::SEPARATE ? 8 : 4) * column) << (8 * k);
            }
            v[i] = x;
        }
    }
};

// Byte address of the cell for slot s of this lane's token, of the table or (BIN) of the bins.  (The bins of SEPARATE
// are 64 KB further, one more than an LDS instruction's offset field holds.)
template <bool BIN, int GH, int B>
__device__ __forceinline__ unsigned code_addr(const Tile<GH, B>& w, const Cols<GH, B>& col, int s)
{
    const u32x4 q = w.lo[s >> 4];
    const int dw = (s >> 2) & 3;
    const unsigned code_word = dw == 0 ? q.x : dw == 1 ? q.y : dw == 2 ? q.z : q.w;
    const unsigned k = s & 3;
    const unsigned sel = 0x0c0c0000u | ((4u + k) << 8) | k;   // {0, 0, code byte k, column byte k}
    unsigned at = __builtin_amdgcn_perm(code_word, col.v[s >> 2], sel);
    if constexpr (B != 8) at |= ((w.hi >> (2 * s)) & 3u) << 6;
    if constexpr (!Lay<GH, B>::SEPARATE) at <<= 1;
    if constexpr (BIN) at |= Lay<GH, B>::BIN_BYTES;
    return at;
}

typedef float pair_f32 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) pair_f32 lds_pair;
typedef __attribute__((address_space(3))) unsigned long long lds_u64;

// (phases, fixed point, the fused step and the walk as in the kernel for one head; m0, l, fx, ... are kept per head)
template <int GH, int C, int B, int NS, bool STEP, bool LAYERS>
__global__ __launch_bounds__(kPairThreads, 4) void decode_pair_kernel(DecodeArgs a)
{
    using F = Lay<GH, B>;
    constexpr int NT = kPairThreads;
    constexpr int K = F::K, R = F::R;
    constexpr int NW = F::NW;           // wavefronts
    constexpr int D = GH * C;           // head_dim
    // tiles in flight per wavefront (about 4 KB)
    constexpr int PF = B == 10 ? 2 : (GH == 16 ? 4 : (GH == 32 ? 2 : 1));
    static_assert(NS % PF == 0 && NS >= PF, "the ring of tiles in flight must divide a chunk");
    constexpr int JPL = 8 / C;          // centroids per 16-byte load
    // groups per chunk of the codebook walk; 64 / GPC neighbouring lanes are on a group and read as
    // many neighbouring 16-byte pieces.  (Measured: four lanes, 64 contiguous bytes, is the
    // optimum; eight -- whole cache lines, but eight lanes on one LDS column and twice the chunks
    // -- is 3 to 10 % slower at every format, two -- all 32 LDS columns in one store, but 32-byte
    // runs -- 2 to 12 %.)
    constexpr int GPC = 16;
    constexpr int LPG = 64 / GPC;
    static_assert(LPG == 4, "lanes_sum<2>");
    constexpr int NCH = GH / GPC;       // chunks of the codebook walk
    constexpr int UNITS = GPC * K / JPL;    // 16-byte loads per chunk
    constexpr int IPT = UNITS / NT;     // ... per thread
    constexpr int KB = IPT < 8 ? IPT : 8;   // ... requested together
    constexpr int KU = IPT / KB <= 2 ? IPT / KB : 1;    // (1024 rows: the batches stay a loop, for registers)
    static_assert(UNITS % NT == 0 && NT % 64 == 0, "thread count must divide the codebook walk");
    extern __shared__ float smem[];
    char* tab = reinterpret_cast<char*>(smem);      // score table and bins, by Lay::cell
    float* slots = smem + F::SLOTS;
    unsigned* sums = reinterpret_cast<unsigned*>(smem + F::SUMS);
    float* scr = smem + F::SCR;
    // fused step: 64-bit (distance, index) minima per group, keys[0..GH) for K, [GH..2GH) for V
    unsigned long long* keys = reinterpret_cast<unsigned long long*>(smem + F::KEYS(D));

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Workgroup -> (sequence, split, query head).  Consecutive workgroups go to consecutive XCDs
    // (8 of them, each with its own L2), so the KV head is made a function of blockIdx % 8 where
    // the head count allows: every workgroup that reads a head's codebooks and code streams then
    // shares one L2 (with grouped queries that is 4 query heads x splits x sequences per head).
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    // layer-batched launch: this workgroup's layer and that layer's tensors
    int bid = blockIdx.x;
    const uint16_t* q_ptr = a.q;
    const uint16_t* xk_new = a.xk_new;
    const uint16_t* xv_new = a.xv_new;
    const uint8_t* k_codes = a.k_codes;
    const uint8_t* v_codes = a.v_codes;
    const uint16_t* k_centroids = a.k_centroids;
    const uint16_t* v_centroids = a.v_centroids;
    uint16_t* out_ptr = a.out;
    float* partials = a.partials;
    if constexpr (LAYERS) {
        const int layer = bid / (a.wgs_per_layer / H);
        bid -= layer * (a.wgs_per_layer / H);
        const LayerPtrsGlobal& lp = reinterpret_cast<const LayerPtrsGlobal*>(a.layers)[layer];
        q_ptr = (const uint16_t*)lp.q;
        xk_new = (const uint16_t*)lp.xk_new;
        xv_new = (const uint16_t*)lp.xv_new;
        k_codes = (const uint8_t*)lp.k_codes;
        v_codes = (const uint8_t*)lp.v_codes;
        k_centroids = (const uint16_t*)lp.k_centroids;
        v_centroids = (const uint16_t*)lp.v_centroids;
        out_ptr = (uint16_t*)lp.out;
        partials += (size_t)layer * a.wgs_per_layer * (D + kPartialHeader);
    }
    const int64_t q_batch_stride = a.q_batch_stride, out_batch_stride = a.out_batch_stride;
    const int seq_len_shift = a.seq_len_shift, seq_len_floor = a.seq_len_floor;
    int hq, split, n;
    if (a.f.n_kv_heads % 8 == 0) {
        const int xcd = bid & 7;
        int r = bid >> 3;
        const int per_xcd = a.f.n_kv_heads >> 3;
        const int hkv_ = xcd + 8 * (r % per_xcd);
        r /= per_xcd;
        const int sets = qper / H;
        hq = hkv_ * qper + r % sets * H;
        r /= sets;
        split = r % a.n_split;
        n = r / a.n_split;
    } else {
        int idx = bid;
        const int sets = a.n_q_heads / H;
        hq = idx % sets * H;
        idx /= sets;
        split = idx % a.n_split;
        n = idx / a.n_split;
    }
    const int hkv = hq / qper;

    int t_n = a.t;
    if (a.seq_lens) t_n = min(max(a.seq_lens[n] - seq_len_shift, seq_len_floor), a.t);
    const int n_tiles = (t_n + kTileTokens - 1) / kTileTokens;
    const int tile0 = split * a.tiles_per_split;
    const int tile1 = min(tile0 + a.tiles_per_split, n_tiles);

    // heads hq and hq + 1, whose rows are neighbours
    float* part = partials + ((size_t)(n * a.n_q_heads + hq) * a.n_split + split) * (D + kPartialHeader);
    const size_t part_head = (size_t)a.n_split * (D + kPartialHeader);
    // (when the launch brought counters; else a merge kernel follows)
    auto count_and_merge = [&] {
        if (!a.merge_counters || !counted_last<D>(a, part, sums, tid)) return;
        const int h = tid / D;              // (a thread per channel and head)
        if (h < H)
            merge_splits<true>(part + h * part_head - (size_t)split * (D + kPartialHeader), a.n_split, D,
                               out_ptr + (size_t)n * out_batch_stride + (size_t)(hq + h) * D, tid % D, D);
    };
    if (tile0 >= tile1) {               // this split lies beyond the sequence: neutral partial
        for (int h = 0; h < H; ++h) {
            if (tid == 0) { partial_store(part + h * part_head, -INFINITY); partial_store(part + h * part_head + 1, 0.f); }
            for (int i = tid; i < D; i += NT) partial_store(part + h * part_head + kPartialHeader + i, 0.f);
        }
        count_and_merge();
        return;
    }

    // fused step: position of the new token, and whether this workgroup's split holds it
    const int pos_new = t_n - 1;
    const int tile_new = pos_new / kTileTokens, u_new = pos_new % kTileTokens;
    const bool has_new = STEP && tile_new >= tile0 && tile_new < tile1;
    if (has_new) {
        if (tid < 2 * GH) keys[tid] = ~0ull;
        lds_barrier();
    }

    // per-lane column constants: the table's, and the same shifted to the bins
    Cols<GH, B> col;
    col.init(lane);

    // this wavefront's tiles: tile0 + wave + k NW, k = 0 .. my_tiles - 1; chunk c holds k = c NS .. c NS + NS - 1
    const int my_tiles = (tile1 - tile0 - wave + NW - 1) / NW;
    const int n_chunks = ((tile1 - tile0 + NW - 1) / NW + NS - 1) / NS;      // of wavefront 0, which has the most tiles
    // The two code streams of this (sequence, KV head).  Contiguous cache: consecutive tiles are
    // TILE_BYTES apart.  Paged cache: lane j holds the page of the j-th tile of the wavefront's
    // current chunk (read one chunk ahead), and a tile sits at base + page * page_bytes.
    const bool paged = a.map.block_table != nullptr;
    const size_t page_bytes = paged ? (size_t)a.f.n_kv_heads * F::TILE_BYTES : 0;
    const size_t stream0 = paged ? (size_t)hkv * F::TILE_BYTES : a.map.tile_index(n, hkv, 0) * F::TILE_BYTES;
    const uint8_t* kbase = k_codes + stream0;
    const uint8_t* vbase = v_codes + stream0;
    auto chunk_pages = [&](int c) {
        int pg = 0;
        const int k = c * NS + lane;
        if (paged && lane < NS && k < my_tiles) pg = a.map.page(n, tile0 + wave + k * NW);
        return pg;
    };
    int pages = chunk_pages(0), pages_next = 0;
    // Request tile i (a compile-time index) of chunk c of a stream.  All of it is scalar
    // arithmetic; the tile's index goes through an opaque copy so that nothing derived from it is
    // kept in registers from one use of the tile to the next (request and use in both streams:
    // that was a pair of scalar registers per tile and condition, and spills).
    const size_t cont_bytes = paged ? 0 : (size_t)F::TILE_BYTES;
    auto request = [&](const uint8_t* base, int c, int i, int pg) {
        int k = c * NS + i;
        asm volatile("" : "+s"(k));
        const bool exists = k < my_tiles;
        const size_t off = (size_t)(unsigned)__builtin_amdgcn_readlane(pg, i) * page_bytes +
                           (size_t)(tile0 + wave + k * NW) * cont_bytes;
        return load_tile_desc<GH, B>(base + (exists ? off : 0), exists, lane);
    };
    // whether tile i of chunk c exists, for the uses (an opaque copy again)
    auto tile_exists = [&](int c, int i) {
        int k = c * NS + i;
        asm volatile("" : "+s"(k));
        return k < my_tiles;
    };
    Tile<GH, B> buf[PF];

    // ---- 1. score table ------------------------------------------------------------------
    // A chunk of the walk is GPC groups; a thread stays on group gl of every chunk.  16-byte piece
    // k of its walk through a group's codebook (centroids j0 .. j0 + JPL - 1, j0 = piece * JPL):
    // the LPG lanes of a group are neighbours and read LPG neighbouring pieces, so the 16 lanes
    // that the memory pipeline takes together read four runs of 64 bytes (with lanes l, l + 16,
    // l + 32, l + 48 on a group, as it first was, they touched 16 lines for 16 bytes each).
    const int gl = (tid / LPG) % GPC;
    auto piece = [&](int k) { return ((tid + k * NT) >> 6) * LPG + (tid % LPG); };
    unsigned xvw[STEP ? NCH : 1][C / 2];            // fused step: this thread's slices of the new value row
    {
        const uint16_t* qh = q_ptr + (size_t)n * q_batch_stride + (size_t)hq * D;
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            const int g = ch * GPC + gl;
            const uint16_t* ck = k_centroids + (size_t)(hkv * GH + g) * K * C;
            unsigned qw[H][C / 2];
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int i = 0; i < C / 2; ++i) qw[h][i] = *reinterpret_cast<const unsigned*>(qh + h * D + g * C + 2 * i);
            // fused step: the new key row against this group's codebook, same walk (the row's
            // words are only requested here; they are converted after the loads below went out)
            unsigned xkw[C / 2];
            float xk[C];
            Nearest knear;
            if (has_new) {
                const size_t xoff = (size_t)n * a.x_new_stride + (size_t)(hkv * GH + g) * C;
#pragma unroll
                for (int i = 0; i < C / 2; ++i) {
                    xkw[i] = *reinterpret_cast<const unsigned*>(xk_new + xoff + 2 * i);
                    xvw[ch][i] = *reinterpret_cast<const unsigned*>(xv_new + xoff + 2 * i);
                }
            }
#pragma unroll(KU)
            for (int k0 = 0; k0 < IPT; k0 += KB) {
                Cent16 raw[KB];
#pragma unroll
                for (int k = 0; k < KB; ++k) raw[k] = load_cent16(ck + (size_t)piece(k0 + k) * 8);
                // the first key tiles are requested behind the first centroids: tile requests must
                // go out as early as possible (the kernel is bound by HBM from its first
                // microsecond), but not in front of the loads the table build waits for
                if (ch == 0 && k0 == 0) {
#pragma unroll
                    for (int i = 0; i < PF; ++i) {
                        buf[i] = request(kbase, 0, i, pages);
                        __builtin_amdgcn_sched_barrier(0);      // keep request order == consumption order
                    }
                    // the bins start at zero (the barrier behind the table build covers these stores)
                    if constexpr (F::SEPARATE) {
                        float4* t4 = reinterpret_cast<float4*>(tab);
#pragma unroll
                        for (int i = tid; i < K * 8 * H; i += NT)
                            t4[(int)(F::BIN_BYTES / 16) + i] = make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                }
                if constexpr (STEP) __builtin_amdgcn_sched_barrier(0);
                if (has_new && k0 == 0) {
#pragma unroll
                    for (int i = 0; i < C / 2; ++i) {
                        const half2_t h = __builtin_bit_cast(half2_t, xkw[i]);
                        xk[2 * i] = (float)h.x;
                        xk[2 * i + 1] = (float)h.y;
                    }
                }
#pragma unroll
                for (int k = 0; k < KB; ++k) {
                    const int j0 = piece(k0 + k) * JPL;
#pragma unroll
                    for (int jj = 0; jj < JPL; ++jj) {
                        float v[H];
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            float dot = 0.f;
#pragma unroll
                            for (int i = 0; i < C / 2; ++i)
                                dot = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, raw[k].w[jj * (C / 2) + i]),
                                                             __builtin_bit_cast(half2_t, qw[h][i]), dot, false);
                            v[h] = dot * a.scale_log2e;
                        }
                        char* dst = tab + F::cell(j0 + jj, g * R);
                        if constexpr (R == 2) *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[0], v[1]);
                        else *reinterpret_cast<float2*>(dst) = make_float2(v[0], v[1]);
                        if (has_new) knear.offer(centroid_distance<C>(xk, &raw[k].w[jj * (C / 2)]), j0 + jj);
                    }
                }
            }
            if (has_new) {
                const unsigned long long kkey = group_lanes_min<LPG>(knear.key());
                if (lane % LPG == 0) lds_min_u64(&keys[g], kkey);
            }
        }
    }
    lds_barrier();

    // fused step: the key codes of the new token are known; the first query head of the KV head
    // stores them (each token owns its 16-byte records, so no other token's bytes are touched)
    const bool writer = has_new && hq % (a.n_q_heads / a.f.n_kv_heads) == 0;
    if (writer)
        store_new_codes<GH, B>(const_cast<uint8_t*>(k_codes) + a.map.tile_index(n, hkv, tile_new) * F::TILE_BYTES, keys, u_new, tid);
    // fused step: the wavefront whose walk meets the new token's tile patches that tile in registers
    // as if the codes just found were already in the cache
    const bool meets_new = has_new && (tile_new - tile0) % NW == wave;
    const NewTokenRecord<GH, B> new_codes{reinterpret_cast<unsigned*>(keys) + NewTokenWords<GH, B>::RECORD};
    if (meets_new) new_codes.build(keys, u_new, lane);

    // ---- 2. the walk: per chunk, scores from the key tiles, then bins from the value tiles ----
    // Fixed point.  A probability is binned as pf = round(2^(s - m0 + fx)): m0 is the maximum of
    // the first chunk, fx an integer.  With (m, l) the running pair of all scores seen so far,
    // the bins of a group then sum to about U = l 2^(m - m0 + fx).  fx starts so that the first
    // chunk's U times the number of chunks lies in [2^29, 2^30); before a later chunk is binned,
    // U including that chunk is predicted from the pair, and if it could pass 2^31.5 every bin
    // (and the running integer sum) is shifted right, rounding to nearest, so that U comes to lie
    // in [2^28, 2^29), and fx drops by the shift.  No bin can overflow 32 bits, and each
    // probability is kept to an absolute error of at most 2^-29 of the softmax denominator.
    constexpr bool EARLY = IPT * NCH <= 8 && KB == IPT;
    Cent16 rawv[EARLY ? NCH : 1][KB];
    unsigned* pf_new = reinterpret_cast<unsigned*>(keys) + NewTokenWords<GH, B>::WEIGHT;
    float m0[H] = {}, m_run[H] = {}, l_run[H] = {}, fxf[H] = {};
    int fx[H] = {};
    unsigned lane_sum[H] = {}, l_carry[H] = {};

    // one key tile: the lane's score, its running pair
    float lane_m[H], lane_l[H];
    struct Scores {
        float s[H];
    };
    Scores sreg[NS];
    auto score_tile = [&](const Tile<GH, B>& w_in, int k, bool turns) {
        Scores score;
        if (turns) take_turns(wave, k);
        const int tile = tile0 + wave + k * NW;
        Tile<GH, B> w = w_in;
        if (meets_new && tile == tile_new) new_codes.patch(w, u_new, lane);
        float acc0[H] = {}, acc1[H] = {};
#pragma unroll
        for (int s = 0; s < GH; s += 2) {
            const unsigned at0 = code_addr<false, GH, B>(w, col, s), at1 = code_addr<false, GH, B>(w, col, s + 1);
            const pair_f32 x0 = *(lds_pair*)(at0), x1 = *(lds_pair*)(at1);
#pragma unroll
            for (int h = 0; h < H; ++h) {
                acc0[h] += x0[h];
                acc1[h] += x1[h];
            }
            // (16 gathers at a time, 32 registers: more spilled)
            if (s % 16 == 14) {
                asm volatile("" : "+v"(acc0[0]), "+v"(acc1[0]), "+v"(acc0[1]), "+v"(acc1[1]));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const int tok = tile * kTileTokens + lane;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            float sv = tok < t_n ? acc0[h] + acc1[h] : -INFINITY;
            // (the sum is formed here, behind its gathers: left free, the compiler sinks the additions of
            // all tiles of a chunk behind the last tile and runs out of registers for the gathered words)
            asm volatile("" : "+v"(sv));
            const float m_new = fmaxf(lane_m[h], sv);
            lane_l[h] = __builtin_fmaf(lane_l[h], __builtin_amdgcn_exp2f(lane_m[h] - m_new), __builtin_amdgcn_exp2f(sv - m_new));
            lane_m[h] = m_new;
            score.s[h] = sv;
        }
        return score;
    };
    // one value tile: the lane's probability in fixed point into the bins of its token's codes
    auto bin_tile = [&](const Tile<GH, B>& w, int k, Scores sv) {
        const int tile = tile0 + wave + k * NW;
        unsigned pf[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const float p = __builtin_amdgcn_exp2f((sv.s[h] - m0[h]) + fxf[h]);
            pf[h] = (unsigned)(p + 0.5f);             // round to nearest
            lane_sum[h] += pf[h];
        }
        // fused step: the new token's value codes are found in the epilogue (the value codebook is
        // loaded there anyway); its weight waits in LDS and joins the bins then
        if (has_new && tile == tile_new && lane == u_new) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
                pf_new[h] = pf[h];
                pf[h] = 0;
            }
        }
        // (no bin reaches 2^32: nothing is carried from one head's half to the other's)
        const unsigned long long both = pf[0] | ((unsigned long long)pf[1] << 32);
#pragma unroll
        for (int s = 0; s < GH; ++s)
            __hip_atomic_fetch_add((lds_u64*)(code_addr<true, GH, B>(w, col, s)), both, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // the value centroids of the epilogue are requested behind the last value tiles, so their
    // latency overlaps the last tiles and the wait for the slowest wavefront (where registers
    // allow: not with 1024 rows)
    auto request_value_centroids = [&] {
        if constexpr (EARLY) {
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
                const uint16_t* cv = v_centroids + (size_t)(hkv * GH + ch * GPC + gl) * K * C;
#pragma unroll
                for (int kk = 0; kk < IPT; ++kk) rawv[ch][kk] = load_cent16(cv + (size_t)piece(kk) * 8);
            }
        }
    };

    // Chunk c.  FULL: all NS tiles of this wavefront exist (always so before the last chunk): the
    // requests run PF tiles ahead through the key tiles, on into the value tiles and on into the
    // next chunk's key tiles, without a condition anywhere.  Otherwise (the wavefront's share of
    // the last chunk is short or empty) the tiles are taken in blocks of PF, blocks without tiles
    // are skipped, and the value tiles are first requested when the key tiles are done.
    auto chunk = [&](int c, auto last_tag, auto full_tag) {
        constexpr bool LAST = decltype(last_tag)::value;
        constexpr bool FULL = decltype(full_tag)::value;
        static_assert(LAST || FULL, "only the last chunk can be short");
        if (paged && !LAST) pages_next = chunk_pages(c + 1);
        const int n_c = my_tiles - c * NS;          // (FULL: >= NS)
        // -- scores.  Every lane also keeps the maximum of its scores and l = sum 2^(s - m) over
        // them (the usual running pair), so that the chunk's pair is known as soon as the
        // wavefronts have exchanged one pair each.
#pragma unroll
        for (int h = 0; h < H; ++h) {
            lane_m[h] = -1e30f;                     // (finite start: a lane without valid tokens stays at l = 0)
            lane_l[h] = 0.f;
        }
        Scores none;
#pragma unroll
        for (int h = 0; h < H; ++h) none.s[h] = -INFINITY;
        constexpr bool kTurns = B == 10 || GH == 64 || (GH == 16 && NS == 8);      // (of a FULL chunk; see take_turns)
        if constexpr (FULL) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                // (the tile exists; the test keeps each tile's arithmetic in a block of its own, which the
                // compiler schedules with far fewer registers than the chunk as one block)
                sreg[i] = tile_exists(c, i) ? score_tile(buf[i % PF], c * NS + i, kTurns) : none;
                // the request PF tiles ahead: a key tile of this chunk, then its first value tiles
                buf[i % PF] = i + PF < NS ? request(kbase, c, i + PF, pages) : request(vbase, c, i + PF - NS, pages);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int ib = 0; ib < NS / PF; ++ib) {
                if (ib * PF < n_c) {                 // (wave-uniform)
#pragma unroll
                    for (int ii = 0; ii < PF; ++ii) {
                        const int i = ib * PF + ii;
                        sreg[i] = tile_exists(c, i) ? score_tile(buf[ii], c * NS + i, false) : none;
                        if (i + PF < NS) buf[ii] = request(kbase, c, i + PF, pages);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
#pragma unroll
                    for (int ii = 0; ii < PF; ++ii) sreg[ib * PF + ii] = none;
                }
            }
#pragma unroll
            for (int ii = 0; ii < PF; ++ii) {
                buf[ii] = request(vbase, c, ii, pages);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (FULL && kTurns) __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const float wave_m = wave_max(lane_m[h]);
            const float wave_l = wave_sum(lane_l[h] * __builtin_amdgcn_exp2f(lane_m[h] - wave_m));
            float* sl = slots + ((c & 1) * H + h) * 2 * NW;
            if (lane == 0) {
                sl[wave] = wave_m;
                sl[NW + wave] = wave_l;
            }
        }
        lds_barrier();              // the chunk's pairs are visible; every bin update of the chunk before is done
        {
            int sh[H] = {};                     // this many bits off the bins
            bool shift = false;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                float m_c, l_c;         // (every chunk holds at least one valid token, so m_c is a score)
                merge_pairs<NW>(slots + ((c & 1) * H + h) * 2 * NW, lane, m_c, l_c);
                if (c == 0) {
                    m0[h] = m_run[h] = m_c;
                    l_run[h] = l_c;
                    fx[h] = fixed_point_exponent(l_c * (float)n_chunks);
                } else if constexpr (F::SEPARATE) {
                    const float m_new = fmaxf(m_run[h], m_c);
                    l_run[h] = l_run[h] * __builtin_amdgcn_exp2f(m_run[h] - m_new) + l_c * __builtin_amdgcn_exp2f(m_c - m_new);
                    m_run[h] = m_new;
                    const float lg_u = __builtin_amdgcn_logf(l_run[h]) + (m_run[h] - m0[h]) + (float)fx[h];
                    if (lg_u >= 31.5f) {
                        sh[h] = (int)floorf(lg_u) - 28;
                        shift = true;
                    }
                }
            }
            if constexpr (F::SEPARATE) {
                if (shift) {                    // (uniform over the workgroup: every thread computes the same)
                    // all wavefronts are between the barrier above and the one below: the bins are quiet
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        const unsigned ws = wave_sum_u32(lane_sum[h]);
                        lane_sum[h] = 0;
                        if (lane == 0) sums[h * NW + wave] = ws;
                    }
                    uint4* b4 = reinterpret_cast<uint4*>(tab);
                    auto half_of = [](int bits) { return bits > 0 && bits < 32 ? 1u << (bits - 1) : 0u; };
                    auto shifted = [&](unsigned v, int bits) { return bits >= 32 ? 0u : (v + half_of(bits)) >> bits; };
                    for (int i = tid; i < 4096; i += NT) {             // 64 KB, 16 bytes at a time
                        uint4* p = b4 + F::BIN_BYTES / 16 + i;
                        uint4 v = *p;
                        v.x = shifted(v.x, sh[0]);
                        v.y = shifted(v.y, sh[1]);
                        v.z = shifted(v.z, sh[0]);
                        v.w = shifted(v.w, sh[1]);
                        *p = v;
                    }
                    lds_barrier();
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        unsigned tot = l_carry[h];
#pragma unroll
                        for (int w = 0; w < NW; ++w) tot += sums[h * NW + w];
                        l_carry[h] = shifted(tot, sh[h]);
                        fx[h] -= sh[h];
                    }
                }
            }
#pragma unroll
            for (int h = 0; h < H; ++h) fxf[h] = (float)fx[h];
        }
        if constexpr (!F::SEPARATE) {           // the table becomes the bins (single chunk)
            float4* t4 = reinterpret_cast<float4*>(tab);
#pragma unroll 4
            for (int i = tid; i < (int)F::TAB_BYTES / 16; i += NT) t4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            lds_barrier();
        }
        // -- bins
        if constexpr (FULL) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                if (tile_exists(c, i)) bin_tile(buf[i % PF], c * NS + i, sreg[i]);
                // the request PF tiles ahead: a value tile of this chunk, then the first key tiles of the next
                if (i + PF < NS) {
                    buf[i % PF] = request(vbase, c, i + PF, pages);
                } else if constexpr (!LAST) {
                    buf[i % PF] = request(kbase, c + 1, i + PF - NS, pages_next);
                } else if (i + PF == NS) {
                    request_value_centroids();
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            const int last_blk = n_c > 0 ? (n_c - 1) / PF : 0;
#pragma unroll
            for (int ib = 0; ib < NS / PF; ++ib) {
                if (ib <= last_blk) {                // (wave-uniform; block 0 always runs)
#pragma unroll
                    for (int ii = 0; ii < PF; ++ii) {
                        const int i = ib * PF + ii;
                        if (tile_exists(c, i)) bin_tile(buf[ii], c * NS + i, sreg[i]);
                        if (i + PF < NS) buf[ii] = request(vbase, c, i + PF, pages);
                        __builtin_amdgcn_sched_barrier(0);
                        if (ii == PF - 1 && ib == last_blk) request_value_centroids();
                    }
                }
            }
        }
        pages = pages_next;
    };
    if constexpr (F::SEPARATE) {
        for (int c = 0; c + 1 < n_chunks; ++c) chunk(c, std::false_type{}, std::true_type{});
    }
    if (my_tiles >= n_chunks * NS) chunk(n_chunks - 1, std::true_type{}, std::true_type{});
    else chunk(n_chunks - 1, std::true_type{}, std::false_type{});

    // ---- 3. epilogue: o = bins . C_V -----------------------------------------------------
    // same walk as the table build; thread-private sums over its centroids of group gl in every
    // chunk, then the four lanes of a group and the wavefronts are added up.
#pragma unroll
    for (int h = 0; h < H; ++h) lane_sum[h] = wave_sum_u32(lane_sum[h]);

    // fused step: encode the new value row against the value codebook (same walk, same registers
    // as the sums below).  A wavefront does this as soon as its own tiles are done, i.e. while it
    // would otherwise wait at the barrier for the slowest one (the minima go to LDS words of
    // their own).
    if (has_new) {
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            float xv[C];
#pragma unroll
            for (int i = 0; i < C / 2; ++i) {
                const half2_t h = __builtin_bit_cast(half2_t, xvw[ch][i]);
                xv[2 * i] = (float)h.x;
                xv[2 * i + 1] = (float)h.y;
            }
            const uint16_t* cv = v_centroids + (size_t)(hkv * GH + ch * GPC + gl) * K * C;
            Nearest vnear;
#pragma unroll(KU)
            for (int k0 = 0; k0 < IPT; k0 += KB) {
                Cent16 rawb[EARLY ? 1 : KB];
                if constexpr (!EARLY) {
#pragma unroll
                    for (int k = 0; k < KB; ++k) rawb[k] = load_cent16(cv + (size_t)piece(k0 + k) * 8);
                }
#pragma unroll
                for (int k = 0; k < KB; ++k) {
                    const int j0 = piece(k0 + k) * JPL;
                    const Cent16& r = EARLY ? rawv[EARLY ? ch : 0][k] : rawb[EARLY ? 0 : k];
#pragma unroll
                    for (int jj = 0; jj < JPL; ++jj) vnear.offer(centroid_distance<C>(xv, &r.w[jj * (C / 2)]), j0 + jj);
                }
            }
            const unsigned long long vkey = group_lanes_min<LPG>(vnear.key());
            if (lane % LPG == 0) lds_min_u64(&keys[GH + ch * GPC + gl], vkey);
        }
    }
    lds_barrier();                                // all bin updates done
    if (lane == 0) {
#pragma unroll
        for (int h = 0; h < H; ++h) sums[h * NW + wave] = lane_sum[h];
    }
    // fused step: the new token's weight joins the bins of the codes just found; store the codes
    if (has_new) {
        if (tid < GH) {
            const unsigned code = (unsigned)(keys[GH + tid] & 0xffffffffu);
#pragma unroll
            for (int h = 0; h < H; ++h) lds_add(F::cell((int)code, tid * R) + F::BIN_BYTES + 4u * h, pf_new[h]);
        }
        if (writer)
            store_new_codes<GH, B>(const_cast<uint8_t*>(v_codes) + a.map.tile_index(n, hkv, tile_new) * F::TILE_BYTES, keys + GH, u_new, tid);
        lds_barrier();
    }

    // one fixed-point unit of the bins, relative to the split's maximum
    float unit[H];
#pragma unroll
    for (int h = 0; h < H; ++h) unit[h] = __builtin_amdgcn_exp2f((m0[h] - m_run[h]) - fxf[h]);
    float acc[NCH][H][C];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int i = 0; i < C; ++i) acc[ch][h][i] = 0.f;
#pragma unroll(KU)
        for (int k0 = 0; k0 < IPT; k0 += KB) {
            if constexpr (!EARLY) {
                const uint16_t* cv = v_centroids + (size_t)(hkv * GH + ch * GPC + gl) * K * C;
#pragma unroll
                for (int k = 0; k < KB; ++k) rawv[0][k] = load_cent16(cv + (size_t)piece(k0 + k) * 8);
            }
            const Cent16 (&raw)[KB] = rawv[EARLY ? ch : 0];
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                const int j0 = piece(k0 + k) * JPL;
#pragma unroll
                for (int jj = 0; jj < JPL; ++jj) {
                    const char* src = tab + F::cell(j0 + jj, (ch * GPC + gl) * R) + F::BIN_BYTES;
                    unsigned cnt[H];
                    if constexpr (R == 2) {
                        const uint4 x = *reinterpret_cast<const uint4*>(src);
                        cnt[0] = x.x + x.z;
                        cnt[1] = x.y + x.w;
                    } else {
                        const uint2 x = *reinterpret_cast<const uint2*>(src);
                        cnt[0] = x.x;
                        cnt[1] = x.y;
                    }
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        const float bin = (float)cnt[h] * unit[h];
#pragma unroll
                        for (int i = 0; i < C / 2; ++i) {
                            const half2_t v = __builtin_bit_cast(half2_t, raw[k].w[jj * (C / 2) + i]);
                            acc[ch][h][2 * i] = __builtin_fmaf(bin, (float)v.x, acc[ch][h][2 * i]);
                            acc[ch][h][2 * i + 1] = __builtin_fmaf(bin, (float)v.y, acc[ch][h][2 * i + 1]);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int i = 0; i < C; ++i) acc[ch][h][i] = lanes_sum<2>(acc[ch][h][i]);
    }
    // per-wave results: scr[64 + (h * NW + wave) * D + channel]
    if (lane % LPG == 0) {
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int i = 0; i < C; ++i) scr[64 + (h * NW + wave) * D + (ch * GPC + gl) * C + i] = acc[ch][h][i];
    }
    lds_barrier();
    unsigned l_fix[H];                              // exact: integer adds
    float l[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        l_fix[h] = l_carry[h];
#pragma unroll
        for (int w = 0; w < NW; ++w) l_fix[h] += sums[h * NW + w];
        l[h] = (float)l_fix[h] * unit[h];
    }
    const bool direct = a.n_split == 1;             // a single split needs no merge
    if (tid == 0 && !direct) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            partial_store(part + h * part_head, m_run[h]);
            partial_store(part + h * part_head + 1, l[h]);
        }
    }
    for (int at = tid; at < H * D; at += NT) {
        const int h = at / D, chn = at % D;
        float o = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) o += scr[64 + (h * NW + w) * D + chn];
        if (direct)
            out_ptr[(size_t)n * out_batch_stride + (size_t)(hq + h) * D + chn] = __builtin_bit_cast(uint16_t, (_Float16)(o / (h == 0 ? l[0] : l[1])));
        else
            partial_store(part + h * part_head + kPartialHeader + chn, o);
    }
    if (!direct) count_and_merge();
}

template <int GH, int C, int B, int NS, bool STEP, bool LAYERS>
cq_status launch_variant(const DecodeArgs& a, hipStream_t stream)
{
    auto kernel = decode_pair_kernel<GH, C, B, NS, STEP, LAYERS>;
    static LdsKernelSetup setup;
    if (setup.ensure(reinterpret_cast<const void*>(kernel)) != hipSuccess) return CQ_ERR_HIP;
    using F = Lay<GH, B>;
    if (!F::SEPARATE && a.tiles_per_split > NS * F::NW) return CQ_ERR_INVALID_ARG;
    const size_t smem = sizeof(float) * (size_t)F::FLOATS(a.f.head_dim, STEP);
    if (smem > 160 * 1024) return CQ_ERR_INVALID_ARG;
    const unsigned grid = (unsigned)(a.batch * (a.n_q_heads / H) * a.n_split) * (unsigned)(a.layers ? a.n_layers : 1);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kPairThreads), smem, stream, a);
    return hipGetLastError() == hipSuccess ? CQ_OK : CQ_ERR_HIP;
}

template <int GH, int C, int B, int NS, bool STEP, bool LAYERS>
cq_status launch_by_length(const DecodeArgs& a, hipStream_t stream)
{
    if (decode_pair_chunk_tiles(a) == NS / 4) return launch_variant<GH, C, B, NS / 4, STEP, LAYERS>(a, stream);
    return launch_variant<GH, C, B, NS / 2, STEP, LAYERS>(a, stream);
}

template <bool STEP, bool LAYERS>
cq_status launch_format(const DecodeArgs& a, hipStream_t stream)
{
    if (a.f.b == 8) {
        if (a.f.gh == 16 && a.f.c == 8) return launch_by_length<16, 8, 8, kChunkTiles8, STEP, LAYERS>(a, stream);
        if (a.f.gh == 32 && a.f.c == 4) return launch_by_length<32, 4, 8, kChunkTiles8, STEP, LAYERS>(a, stream);
        if (a.f.gh == 64 && a.f.c == 2) return launch_by_length<64, 2, 8, kChunkTiles8, STEP, LAYERS>(a, stream);
    } else if (a.f.b == 10 && a.f.gh == 16 && a.f.c == 8) {
        return launch_by_length<16, 8, 10, kChunkTiles10, STEP, LAYERS>(a, stream);
    }
    return CQ_ERR_UNSUPPORTED;
}

}  // namespace

// An even number of query heads per KV head, and enough workgroups: one runs per CU, so fewer than 256 leave CUs idle
// that the kernel for one head uses, and with byte codes a last round of workgroups that fills less than its share
// costs more than the pairs save (32 / 8 heads, one head -> two: 1.25 rounds, 20 x 2000, CQ-8c8b 14.7 -> 19.9 us, CQ-4c8b 20.8 ->
// 24.0; 1.5 rounds, 24 x 3000, step of CQ-4c8b 30.9 -> 33.7; 1.75 rounds, 28 x 4000, CQ-8c8b 25.2 -> 25.4, CQ-4c8b 37.8 -> 32.7, and 28 x
// 16000 64.9 -> 62.4, 110.7 -> 91.6).  CQ-8c10b gains in nearly all of them (17 x 2000 28.0 -> 29.1, 17 x 16000 76.5 -> 71.6, 20 x 2000 28.9 ->
// 29.4, 20 x 16000 78.2 -> 72.0, 24 x 2000 30.3 -> 29.7, 36 x 2000 45.4 -> 43.5): of its codebooks, 256 KB each, a workgroup reads
// half as much per head.  (Calls of CQ-8c8b and CQ-4c8b with heads in fours are offered to cq_decode_quad.hip first, which takes those
// byte-code sizes above; the rule is for two or six heads per KV head as it was for four.  Of a layer-batched launch the layer
// decides, so that its results are those of the layers' own calls.)
bool decode_takes_pairs(const DecodeArgs& a)
{
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    const int64_t wgs = (int64_t)a.batch * (a.n_q_heads / H) * a.n_split, rounds = (wgs + 255) / 256;
    if (qper % H != 0 || wgs < 256) return false;
    return a.f.b == 10 || wgs * 20 >= rounds * 256 * 17;
}

// (twice the wavefronts: half the tiles per wavefront and chunk, of two heads each, so as many score registers)
int decode_pair_chunk_tiles(const DecodeArgs& a)
{
    const int full = (a.f.b == 10 ? kChunkTiles10 : kChunkTiles8) / H, nw = kDecodeWaves * H;
    return (a.tiles_per_split + nw - 1) / nw <= full / 2 ? full / 2 : full;
}

cq_status launch_decode_pair(const DecodeArgs& a, hipStream_t stream)
{
    if (a.layers) return launch_format<true, true>(a, stream);
    return a.xk_new ? launch_format<true, false>(a, stream) : launch_format<false, false>(a, stream);
}

}  // namespace cq
