// Causal attention of the last m tokens of each sequence over its packed CQ cache (a prefill
// chunk, or the verification step of speculative decoding), for gfx950.  Eq. 1 of the paper once
// per query token; the cache already holds the codes of the m tokens.
//
// With many queries per (sequence, KV head) the per-query lookup tables of the decode kernel
// no longer fit on chip and the path becomes a dense contraction, so this one is built on the
// matrix cores: a workgroup (8 wavefronts) owns up to 256 query rows of one KV head (query
// tokens x the query heads that share the KV head), walks the context in 64-token tiles, turns
// each tile's codes back into fp16 keys and values ONCE in LDS (centroid gathers from the
// L2-resident codebooks), and every wavefront runs a flash-attention step on its 32 rows:
//     S^T = K Q^T      v_mfma_f32_32x32x16_f16, A = keys of 32 tokens (LDS), B = queries (registers)
//     online softmax   each lane owns ONE query (a column of S^T): running maximum, sum and the
//                      rescaling of its output column are lane-local
//     O^T += V^T P^T   A = values (LDS, transposed by the read), B = the probabilities just computed,
//                      scaled by 2^12 and split into two fp16 numbers (high and low part: 22
//                      bits; one fp16 alone leaves errors of 1e-5 of the largest output element,
//                      too much for the small ones); fp32 accumulation
// HBM traffic is the codes, read once per workgroup.  Three things take about the same time: the
// matrix cores (rotated keys: 128 products per SIMD and 64-token tile, 4224 clocks), the LDS reads that
// feed them (4600 clocks per CU) and the vector ALU (4900 clocks per SIMD); a tile takes 7500, as two wavefronts
// per SIMD overlap them only in part.  Measured (CQ-8c8b, 32 / 8 heads, 500 rotated query tokens of 2
// sequences x 9001): 384 -> 333 us; 4 x 512 query tokens at 8192, 32 heads: 741 -> 617 us rotated,
// 530 -> 490 us not.  What gave it: straight instruction streams in which products and vector work
// alternate, operands read a group ahead, the queries' loads waited for before the loop, gathers and
// rotation a tile ahead of their use, values kept token by token and transposed by the read, and
// wavefronts that lag before those that lead.  Long contexts with few rows are split over workgroups and
// merged by the decode path's merge kernel (same (m, l, o) partials).
#include "cq_lds_gather.hpp"

namespace cq {
namespace {

typedef float float16_t __attribute__((ext_vector_type(16)));

// 8 wavefronts x 32 query rows per workgroup (one workgroup per CU), or 4 x 32 where a KV head has
// no more than 128 rows (two workgroups per CU then)
constexpr int kKsStride = 272;                    // bytes per token row of the key tile (256 + 16: conflict-free 16-byte reads)
constexpr int kKsBytes = kTileTokens * kKsStride; // 17408
// The value tile has a token's 128 channels in a row too, its four 64-byte quarters exchanged by the token's two
// low bits: the transposing read takes a quarter of four tokens at a time, which then lie in different banks.
constexpr int kVsStride = 256;
constexpr int kVsBytes = kTileTokens * kVsStride; // 16384
// a stage: the key tile, the value tile and (rotated keys only) the low parts of the key tile
constexpr int kStageBytes(bool rope) { return kKsBytes + kVsBytes + (rope ? kKsBytes : 0); }
constexpr unsigned kRawBase(bool rope) { return 2 * kStageBytes(rope); }     // behind the two stages: the raw code tiles (K, V) of two tiles
constexpr unsigned kAngleBytes = 64 * kTileTokens * 8;                       // behind those (rotated keys): cos / sin per pair and token of a tile
typedef __attribute__((address_space(3))) u32x4 lds_q;

__device__ __forceinline__ half8_t lds_half8(unsigned byte_addr)
{
    return *(__attribute__((address_space(3))) half8_t*)(byte_addr);
}
// two numbers as fp16 plus what fp16 leaves of them
__device__ __forceinline__ void split_pair(float x, float y, unsigned& high, unsigned& low)
{
    const half2_t h = __builtin_convertvector(float2_t{x, y}, half2_t);
    float minus = -1.f;                 // (opaque: as a product the difference is one instruction with its conversions)
    asm("" : "+s"(minus));
    half2_t l;
    l.x = (_Float16)__builtin_fmaf((float)h.x, minus, x);
    l.y = (_Float16)__builtin_fmaf((float)h.y, minus, y);
    high = __builtin_bit_cast(unsigned, h);
    low = __builtin_bit_cast(unsigned, l);
}
// the larger of lane i's and lane (i ^ 32)'s value
__device__ __forceinline__ float half_wave_max(float x)
{
    const unsigned u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Codes of 64 tokens -> fp16 keys and values [token][channel] in LDS.
// The codes of a tile first go to LDS as they are (request_codes / store_codes: one 16-byte record per
// thread).  Then thread (token u = tid % 64, wavefront e = tid / 64) expands groups
// e Gh/NW .. (e + 1) Gh/NW - 1 of its token: the code of group g sits in slot (g - u) mod Gh of the
// token's record.  A wavefront thus gathers from ONE group's centroids at a time: its 64 lanes
// touch the 8 to 32 cache lines of that group's table instead of 64 lines of 64 tables, which is
// what the texture path charges for.  Neighbouring groups of one thread also make its stores 16
// bytes wide for every format.
//
// ROPE (keys cached before the rotary position embedding): thread (u, e) takes half as many
// neighbouring groups from each half of the head instead, so that it holds both halves of its channel
// pairs (channel i of the head is rotated with channel i + 64, i.e. group g with group g + Gh/2), and
// rotate() turns the pairs to the token's position before the keys go to LDS: once per (tile, KV
// head), for all query rows of the workgroup.
template <int GH, int C, int NW, int B, bool ROPE>
struct Dequant {
    static constexpr int GPT = GH / NW;                 // groups per thread
    static_assert(!ROPE || GPT % 2 == 0, "a thread holds both groups of a pair");
    static constexpr int NP = ROPE ? GPT / 2 * C : 1;   // channel pairs per thread
    float2 ts[NP];                                      // ROPE: cos / sin of (first position of the tile * theta) of this thread's pairs
    // ROPE: low parts of the rotated keys.  A rotated key is kept as the sum of two fp16 numbers
    // (22 bits): rounded to one, its error of 2^-11 reaches the scores and leaves 4e-4 of a
    // row's largest output element, which fails the 2e-3 bar on the small elements
    unsigned kwl[GPT][C / 2];
    __device__ __forceinline__ static int group(int e, int gi)
    {
        return ROPE ? (gi < GPT / 2 ? 0 : GH / 2) + e * (GPT / 2) + gi % (GPT / 2) : e * GPT + gi;
    }
    static constexpr int K = 1 << B;                    // centroids per group
    static constexpr int TILE = kTileTokens * GH * B / 8;   // bytes of one tile's codes (b = 10: low bytes, then high-bit words)
    static constexpr int LOADERS = TILE / 16;           // threads that carry one record of K and one of V
    static constexpr int RAW_STAGE = 2 * TILE;          // K tile, V tile
    static_assert(LOADERS <= NW * 64, "one record per thread");
    struct Codes {
        u32x4 k, v;
    };
    Codes raw;                                          // 16-byte records of codes on their way to LDS
    unsigned kw[GPT][C / 2], vw[GPT][C / 2];            // the centroids of this thread's (token, group) pairs

    __device__ __forceinline__ static Codes request_codes(const uint8_t* ktile, const uint8_t* vtile, int tid)
    {
        Codes c = {};
        if (tid < LOADERS) {
            c.k = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ktile) + tid);
            c.v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vtile) + tid);
        }
        return c;
    }
    __device__ __forceinline__ static void store_codes(const Codes& c, unsigned k_slot, unsigned v_slot, int tid)
    {
        if (tid < LOADERS) {
            *(lds_q*)(k_slot + (unsigned)tid * 16) = c.k;
            *(lds_q*)(v_slot + (unsigned)tid * 16) = c.v;
        }
    }

    // this thread's codes from the raw tile, and the request for their centroids (L2-resident codebooks)
    unsigned code[GPT];
    __device__ __forceinline__ void read_codes(unsigned raw, int tid)
    {
        typedef __attribute__((address_space(3))) uint8_t lds_b;
        const int u = tid & 63, e = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
        for (int gi = 0; gi < GPT; ++gi) {
            const unsigned slot = (unsigned)(group(e, gi) - u) & (unsigned)(GH - 1);
            code[gi] = *(lds_b*)(raw + (slot >> 4) * 1024 + (unsigned)u * 16 + (slot & 15));
            if constexpr (B == 10) {        // bits [2 s + 1 : 2 s] of the token's high-bit word
                typedef __attribute__((address_space(3))) unsigned lds_w;
                code[gi] |= ((*(lds_w*)(raw + (unsigned)(kTileTokens * GH) + (unsigned)u * 4) >> (2 * slot)) & 3u) << 8;
            }
        }
    }
    // (not `wanted`: zeros, not the old contents, which would occupy their registers until here)
    __device__ __forceinline__ void request(unsigned (&w)[GPT][C / 2], const uint16_t* c_head, int tid, bool wanted) const
    {
        const int e = __builtin_amdgcn_readfirstlane(tid >> 6);
        if (wanted) {
#pragma unroll
            for (int gi = 0; gi < GPT; ++gi) {
                const unsigned* src = reinterpret_cast<const unsigned*>(c_head + ((size_t)group(e, gi) * K + code[gi]) * C);
#pragma unroll
                for (int i = 0; i < C / 2; ++i) w[gi][i] = src[i];
            }
        } else {
#pragma unroll
            for (int gi = 0; gi < GPT; ++gi)
#pragma unroll
                for (int i = 0; i < C / 2; ++i) w[gi][i] = 0;
        }
    }
    __device__ __forceinline__ void gather(unsigned (&w)[GPT][C / 2], unsigned raw, const uint16_t* c_head, int tid, bool wanted)
    {
        read_codes(raw, tid);
        request(w, c_head, tid, wanted);
    }

    // ROPE: the angle of a rotation is the sum of two: u theta_i per lane, whose cos / sin lie in LDS ([pair][lane]),
    // and 64 tile theta_i, the same for the wavefront (read in the constant address space, i.e. through the scalar
    // cache: the table is older than this kernel)
    __device__ __forceinline__ void request_tile_angles(const float2* tile_tab, int tile, int tid)
    {
        if constexpr (ROPE) {
            const int e = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                typedef const __attribute__((address_space(4))) float* scalar_floats;
                const scalar_floats t = (scalar_floats)(tile_tab + (size_t)tile * 64 + e * NP + p);
                ts[p] = make_float2(t[0], t[1]);
            }
        }
    }
    struct Angles {
        float2 c0, c1;
    };
    __device__ __forceinline__ static Angles lane_angles(unsigned table, int tid, int q)
    {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        typedef __attribute__((address_space(3))) f32x2 lds_f2;
        const unsigned at = table + (unsigned)(__builtin_amdgcn_readfirstlane(tid >> 6) * NP + 2 * q) * 512 + (unsigned)(tid & 63) * 8;
        const f32x2 x = *(lds_f2*)at, y = *(lds_f2*)(at + 512);
        return {make_float2(x.x, x.y), make_float2(y.x, y.y)};
    }
    // the same from the table in memory
    __device__ __forceinline__ static Angles table_angles(const float2* lane_tab, int tid, int q)
    {
        const float2* t = lane_tab + (size_t)(__builtin_amdgcn_readfirstlane(tid >> 6) * NP + 2 * q) * 64 + (tid & 63);
        return {t[0], t[64]};
    }
    // rotate pairs 2 q and 2 q + 1 of the gathered keys:
    // (k_i, k_{i+64}) -> (k_i cos - k_{i+64} sin, k_{i+64} cos + k_i sin), fp32, then two fp16 parts
    __device__ __forceinline__ void rotate(const Angles& lane_part, int q)
    {
        if constexpr (ROPE) {
            const int gi = q / (C / 2), i = q % (C / 2);
            auto sum = [](float2 t, float2 l) { return make_float2(t.x * l.x - t.y * l.y, t.y * l.x + t.x * l.y); };
            const float2 c0 = sum(ts[2 * q], lane_part.c0), c1 = sum(ts[2 * q + 1], lane_part.c1);
            const half2_t lo = __builtin_bit_cast(half2_t, kw[gi][i]), hi = __builtin_bit_cast(half2_t, kw[gi + GPT / 2][i]);
            const float fl0 = (float)lo.x * c0.x - (float)hi.x * c0.y, fh0 = (float)hi.x * c0.x + (float)lo.x * c0.y;
            const float fl1 = (float)lo.y * c1.x - (float)hi.y * c1.y, fh1 = (float)hi.y * c1.x + (float)lo.y * c1.y;
            split_pair(fl0, fl1, kw[gi][i], kwl[gi][i]);
            split_pair(fh0, fh1, kw[gi + GPT / 2][i], kwl[gi + GPT / 2][i]);
            // (here, between the products, not behind them)
            asm volatile("" : "+v"(kw[gi][i]), "+v"(kwl[gi][i]), "+v"(kw[gi + GPT / 2][i]), "+v"(kwl[gi + GPT / 2][i]));
        }
    }
    static constexpr int kRotations = ROPE ? GPT / 2 * (C / 2) : 0;

    // the thread's channels in 16-byte pieces (eight channels; its groups lie side by side, in each half of the head
    // for rotated keys), the values first
    static constexpr int PIECES = GPT * C / 8;
    __device__ __forceinline__ static int first_channel(int e, int q)
    {
        return ROPE ? (q < PIECES / 2 ? 0 : 64) + e * (GPT / 2 * C) + 8 * (q % (PIECES / 2)) : e * (GPT * C) + 8 * q;
    }
    __device__ __forceinline__ static u32x4 piece(const unsigned (&w)[GPT][C / 2], int q)
    {
        constexpr int H = C / 2;
        return u32x4{w[(4 * q) / H][(4 * q) % H], w[(4 * q + 1) / H][(4 * q + 1) % H], w[(4 * q + 2) / H][(4 * q + 2) % H],
                     w[(4 * q + 3) / H][(4 * q + 3) % H]};
    }
    __device__ __forceinline__ void store_values(unsigned stage, int tid) const
    {
        const int u = tid & 63, e = __builtin_amdgcn_readfirstlane(tid >> 6);
        const unsigned row = stage + kKsBytes + (unsigned)u * kVsStride;
#pragma unroll
        for (int q = 0; q < PIECES; ++q) *(lds_q*)(row + ((unsigned)(first_channel(e, q) * 2) ^ ((unsigned)(u & 3) << 6))) = piece(vw, q);
    }
    __device__ __forceinline__ void store_keys(unsigned stage, int tid) const
    {
        const int u = tid & 63, e = __builtin_amdgcn_readfirstlane(tid >> 6);
        const unsigned row = stage + (unsigned)u * kKsStride;
#pragma unroll
        for (int q = 0; q < PIECES; ++q) {
            *(lds_q*)(row + (unsigned)(first_channel(e, q) * 2)) = piece(kw, q);
            if constexpr (ROPE) *(lds_q*)(row + (unsigned)(kKsBytes + kVsBytes + first_channel(e, q) * 2)) = piece(kwl, q);
        }
    }
};

// 8 wavefronts are two per SIMD; of the workgroups of 4, two fit on a CU by their LDS but for rotated keys and
// the code tiles of CQ-2c8b: those take the registers of two wavefronts
constexpr int chunk_waves_per_simd(int c, int nw, bool rope) { return nw == 4 && (rope || c == 2) ? 1 : 2; }

// SHORT: pieces of the context of up to kShortTiles tiles, without the look-ahead of the pipeline, whose registers
// (the form of four wavefronts spills some) and prologue such a call does not repay.  Not rotated, pipeline / this:
// CQ-8c8b 64 x 64 tokens over 64: 39.6 / 35.3 us, 40 x 70 over 100: 36.4 / 32.1, 16 x 100 over 190: 20.2 / 18.7,
// CQ-8c10b 43.4 / 37.5, 41.6 / 36.5 and 24.3 / 24.2; over four tiles the pipeline is ahead.  Rotated keys, whose
// pipeline repays itself from two tiles on: CQ-8c8b 64 x 64 over 64: 66.2 / 64.9.
constexpr int kShortTiles(bool rope) { return rope ? 1 : 3; }

template <int GH, int C, int NW, int B, bool ROPE, bool SHORT>
__global__ __launch_bounds__(NW * 64, chunk_waves_per_simd(C, NW, ROPE)) void chunk_attention_kernel(ChunkArgs a)
{
    constexpr int kRowsPerWg = NW * 32;
    constexpr unsigned kRawStageBytes = Dequant<GH, C, NW, B, ROPE>::RAW_STAGE;
    using F = Fmt<GH, B>;
    constexpr int D = 128;
    static_assert(GH * C == D, "head_dim 128");
    extern __shared__ float smem[];
    (void)smem;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rc = lane & 31, kh = lane >> 5;

    // workgroup -> (sequence, KV head, block of 128 query rows, context split)
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    const int rows_total = a.m * qper;                      // row r = (query token r / qper, query head r % qper)
    const int row_blocks = (rows_total + kRowsPerWg - 1) / kRowsPerWg;
    int idx = blockIdx.x;
    const int hkv = idx % a.f.n_kv_heads;
    idx /= a.f.n_kv_heads;
    const int rb = idx % row_blocks;
    idx /= row_blocks;
    const int split = idx % a.n_split;
    const int n = idx / a.n_split;

    int t_n = a.t;
    if (a.seq_lens) t_n = min(max(a.seq_lens[n], a.m), a.t);
    const int pos0 = t_n - a.m;                             // position of query token 0

    // this lane's query row
    const int row = rb * kRowsPerWg + wave * 32 + rc;
    const bool valid = row < rows_total;
    const int row_c = valid ? row : rows_total - 1;
    const int j = row_c / qper, hq = hkv * qper + row_c % qper;
    const int pos = pos0 + j;
    // (rows ascend with the lane: the wavefront's earliest position is its first lane's)
    const int pos_first = __builtin_amdgcn_readfirstlane(pos);
    // tiles this workgroup needs: up to the position of its last row, within its split
    const int last_row = min(rb * kRowsPerWg + kRowsPerWg, rows_total) - 1;
    const int tiles_needed = (pos0 + last_row / qper) / kTileTokens + 1;
    const int tile0 = split * a.tiles_per_split;
    const int tile1 = min(tile0 + a.tiles_per_split, tiles_needed);
    // the wavefront's own last tile (rows of later wavefronts reach further)
    const int wave_last_row = min(rb * kRowsPerWg + wave * 32 + 31, rows_total - 1);
    const int wave_tiles = (pos0 + wave_last_row / qper) / kTileTokens + 1;


    // queries: B operand of S^T = K Q^T, lane (rc, kh) holds Q[row][16 s + 8 kh .. + 7] for the 8 steps
    half8_t qreg[8];
    {
        const uint16_t* qrow = a.q + (((size_t)n * a.m + j) * a.n_q_heads + hq) * D;
#pragma unroll
        for (int s = 0; s < 8; ++s) qreg[s] = *reinterpret_cast<const half8_t*>(qrow + 16 * s + 8 * kh);
    }
    // A negative scale turns the queries' signs, so that the largest product is the largest score; a scale
    // of zero stands for one so small that every weight is 1 (0 times a masked -infinity is no number).
    const float scale = a.scale_log2e == 0.f ? 1e-37f : fabsf(a.scale_log2e);

    const uint16_t* ck_head = a.k_centroids + (size_t)hkv * GH * F::K * C;
    const uint16_t* cv_head = a.v_centroids + (size_t)hkv * GH * F::K * C;
    float16_t o[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[cb][i] = 0.f;
    float ref = -INFINITY, l_run = 0.f;                     // probabilities and their sum are relative to 2^ref

    // One tile of this wavefront, in straight lines of vector and matrix instructions so that the two
    // pipes overlap within the wavefront: while the scores of tokens 32 .. 63 are multiplied, the vector
    // ALU turns those of tokens 0 .. 31 into probabilities, and those of 32 .. 63 while the values of
    // 0 .. 31 are; the rotation of the next tile's keys and its stores go with the last products.  The
    // operands are read from LDS a group of four products ahead.
    constexpr int kParts = ROPE ? 2 : 1;                    // fp16 parts of a key
    constexpr int kGroups = 2 * kParts;                     // groups of four products per 32-token block
    float16_t acc[2];
    float bmax_of[2], alpha_of[2];
    u32x4 ph[2][2], pl[2][2];                               // p = ph + pl to 22 bits
    half8_t kf[2][4];
    auto read_keys = [&](unsigned stage, int g) {           // group g of the tile: block, part, half of the head
        const int tb = g / kGroups, part = g % kGroups / 2, half = g & 1;
        const unsigned krow = stage + (unsigned)(tb * 32 + rc) * kKsStride + (unsigned)kh * 16 + part * (kKsBytes + kVsBytes) + half * 128;
#pragma unroll
        for (int i = 0; i < 4; ++i) kf[g & 1][i] = lds_half8(krow + 32 * i);
    };
    auto multiply_key = [&](int g, int i) {
        const int tb = g / kGroups;
        acc[tb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[g & 1][i], qreg[(g & 1) * 4 + i], acc[tb], 0, 0, 0);
    };
    // softmax of a block in ten slices: the maximum; what follows from it; two probabilities in each of the others.
    // acc[tb][i] is token 8 (i / 4) + 4 kh + i % 4 of the block, query rc
    float psum_of[2], shift_of[2];
    bool large = false;                                     // (set below: see scores_may_be_large)
    float mult = scale, early = 1.f, lead = 10.f;
    auto mask = [&](int tile, int tb) {                     // a tile on the causal diagonal of some query of this wavefront
        if (large || tile * kTileTokens + kTileTokens - 1 > pos_first) {
            const int tok0 = tile * kTileTokens + tb * 32 + 4 * kh;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tb][i] = tok0 + 8 * (i >> 2) + (i & 3) <= pos ? acc[tb][i] * early : -INFINITY;
        }
    };
    auto softmax_slice = [&](int tb, int k) {
        if (k == 0) {
            float b = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; ++i) b = fmaxf(b, acc[tb][i]);
            bmax_of[tb] = b;
        } else if (k == 1) {
            const float ref_new = fmaxf(ref, __builtin_fmaf(half_wave_max(bmax_of[tb]), mult, -lead));
            shift_of[tb] = ref_new == -INFINITY ? 0.f : ref_new;        // nothing visible yet: all weights 0
            alpha_of[tb] = __builtin_amdgcn_exp2f(ref - shift_of[tb]);
            ref = ref_new;
            psum_of[tb] = 0.f;
        } else if (k < 10) {
            const int i = 2 * (k - 2);
            const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[tb][i], mult, -shift_of[tb]));
            const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[tb][i + 1], mult, -shift_of[tb]));
            psum_of[tb] += p0;
            psum_of[tb] += p1;
            unsigned hi, lo;
            split_pair(p0, p1, hi, lo);
            asm volatile("" : "+v"(hi), "+v"(lo));          // here, not behind the products
            ph[tb][i >> 3][i >> 1 & 3] = hi;
            pl[tb][i >> 3][i >> 1 & 3] = lo;
        }
    };
    auto rescale = [&](int tb) {
        if (__builtin_amdgcn_ballot_w64(alpha_of[tb] != 1.f) != 0) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[cb][i] *= alpha_of[tb];
        }
    };
    // O^T += V^T P^T: contraction index (kh, i) of step t is token 16 t + 8 (i / 4) + 4 kh + i % 4 of the block
    half8_t av[2][4];
    // (the transposing read: lane 4 k + q of 16 addresses channels 4 q .. 4 q + 3 of the k-th of four tokens and
    // receives channel 4 k + q of all four)
    const unsigned vlane = (unsigned)(4 * kh + (lane >> 2 & 3)) * kVsStride + ((unsigned)(lane >> 2 & 3) << 6) + ((unsigned)lane & 16) * 2 + (lane & 3) * 8;
    auto read_values = [&](unsigned stage, int tb, int t) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const unsigned vrow = stage + kKsBytes + (vlane ^ ((unsigned)cb << 6)) + (unsigned)(tb * 32 + 16 * t) * kVsStride;
            const half4_t v0 = lds_transposed(vrow), v1 = lds_transposed(vrow + 8 * kVsStride);
            av[t][cb] = half8_t{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
        }
    };
    auto multiply_value = [&](int tb, int k) {              // the 16 products of a block
        const int t = k >> 3, cb = k & 3;
        o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[t][cb], __builtin_bit_cast(half8_t, (k & 4) ? pl[tb][t] : ph[tb][t]), o[cb], 0, 0, 0);
    };
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

    // Software pipeline over the tiles.  While tile k is multiplied, the keys of tile k + 1 are rotated (behind the
    // scores of tokens 0 .. 31) and stored, its values' centroids come from L2 (requested behind them, stored at the
    // end), the centroids of the keys of tile k + 2 are requested (behind the last products), and the codes of the
    // keys of tile k + 3 and the values of tile k + 2 are on their way from HBM: the keys run a tile ahead, so that
    // the gathers, 2048 clocks of the path from L2 per tile, are spread over all of it.
    using D_ = Dequant<GH, C, NW, B, ROPE>;
    D_ dq;
    constexpr unsigned kTileRaw = D_::TILE;
    auto k_slot = [&](int t) { return kRawBase(ROPE) + (unsigned)((t - tile0) & 1) * kRawStageBytes; };
    auto v_slot = [&](int t) { return k_slot(t) + kTileRaw; };
    auto stage_of = [&](int t) { return (unsigned)((t - tile0) & 1) * kStageBytes(ROPE); };
    // (tiles behind the last one stand for it where only an address is made of them)
    auto clamped = [&](int t) { return min(t, tile1 - 1); };
    constexpr unsigned kAngles = kRawBase(ROPE) + 2 * kRawStageBytes;

    size_t v_index = 0;                                     // tile index (of both code arrays) of tile + 2
    auto load_codes = [&](int tile) {                       // codes: keys of tile + 3, values of tile + 2
        if (tile + 2 >= tile1) {
            dq.raw = {};                                    // (not the old contents: they would stay in registers until here)
            return;
        }
        const size_t k_index = a.map.tile_index(n, hkv, clamped(tile + 3));
        dq.raw = D_::request_codes(a.k_codes + k_index * F::TILE_BYTES, a.v_codes + v_index * F::TILE_BYTES, tid);
        v_index = k_index;
    };
    auto end_tile = [&](int tile) {
        if (tile + 2 < tile1) D_::store_codes(dq.raw, k_slot(tile + 3), v_slot(tile + 2), tid);
        dq.request_tile_angles(a.rope_tile_tab, clamped(tile + 2), tid);
        lds_barrier();
    };
    auto rotate_keys = [&] {
#pragma unroll
        for (int q = 0; q < D_::kRotations; ++q) dq.rotate(D_::lane_angles(kAngles, tid, q), q);
    };

    const bool paced = tile1 - tile0 > 8;
    auto multiply_tile = [&](int tile) {
        const unsigned stage = stage_of(tile), next_stage = stage_of(tile + 1);
        typename D_::Angles angles[2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tb][i] = 0.f;
        // The priority falls from phase to phase, so that of the two wavefronts of a SIMD the one that lags goes
        // first: left to the age of the wavefront, one ran ahead and waited at the barrier for a third of the tile.
        // (Not over a few tiles, where another workgroup's prologue would be what waits: CQ-8c8b, 40 x 70 tokens
        // over 100, 39.9 us without and 42.9 with.)
        if (paced) __builtin_amdgcn_s_setprio(3);
        read_keys(stage, 0);
        if constexpr (ROPE) angles[0] = D_::lane_angles(kAngles, tid, 0);
#pragma unroll
        for (int g = 0; g < 2 * kGroups; ++g) {
            if (g == kGroups) {
                if (tile + 1 < tile1) dq.store_keys(next_stage, tid);
                load_codes(tile);                           // (behind the wait for the keys' centroids, before the values')
                mask(tile, 0);
                if (paced) __builtin_amdgcn_s_setprio(2);
            }
            if (g == kGroups - 1) dq.read_codes(v_slot(tile + 1), tid);
            if (g + 1 < 2 * kGroups) read_keys(stage, g + 1);
            else read_values(stage, 0, 0);
            fence();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                multiply_key(g, i);
                if (g == kGroups && i == 0) dq.request(dq.vw, cv_head, tid, tile + 1 < tile1);
                if (ROPE && g < kGroups) {                  // the next tile's keys behind the first products
                    constexpr int per = 16 / (D_::kRotations > 0 ? D_::kRotations : 16);
                    const int idx = 4 * g + i, q = idx / per;
                    if (idx % per == per / 2 && q + 1 < D_::kRotations) angles[(q + 1) & 1] = D_::lane_angles(kAngles, tid, q + 1);
                    if (idx % per == per - 1) dq.rotate(angles[q & 1], q);
                }
                if (g >= kGroups) {
                    constexpr int per = ROPE ? 2 : 1;       // 16 or 8 products for seven slices
                    const int k = (4 * (g - kGroups) + i) / per - (ROPE ? 1 : 0);
                    if ((4 * (g - kGroups) + i) % per == 0 && k >= 0 && k < 7) softmax_slice(0, k);
                }
                fence();
            }
        }
        mask(tile, 1);
        rescale(0);
        if (paced) __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (k == 4) read_values(stage, 0, 1);
            if (k == 12) read_values(stage, 1, 0);
            if (k == 14) dq.read_codes(k_slot(tile + 2), tid);
            fence();
            multiply_value(0, k);
            if (k < 6 && k % 2 == 0) softmax_slice(0, 7 + k / 2);      // the rest of block 0's: tokens of the second half
            if (k >= 5 && k < 12) softmax_slice(1, k - 5);
        }
        l_run = __builtin_fmaf(l_run, alpha_of[0], psum_of[0]);
        fence();
        rescale(1);
        if (paced) __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (k == 4) read_values(stage, 1, 1);
            fence();
            multiply_value(1, k);
            if (k == 0) dq.request(dq.kw, ck_head, tid, tile + 2 < tile1);
            if (k < 6 && k % 2 == 0) softmax_slice(1, 7 + k / 2);
        }
        l_run = __builtin_fmaf(l_run, alpha_of[1], psum_of[1]);
        if (tile + 1 < tile1) dq.store_values(next_stage, tid);
    };

    // (The squares of the queries' norms are the diagonal of Q Q^T, and none of its elements is larger: products on
    // the idle matrix cores, where the first tile's centroids are waited for.  As vector instructions in front of the
    // loop they cost 1 % of a call over five tiles.)
    auto bound_scores = [&] {
        float16_t g;
#pragma unroll
        for (int i = 0; i < 16; ++i) g[i] = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) g = __builtin_amdgcn_mfma_f32_32x32x16_f16(qreg[s], qreg[s], g, 0, 0, 0);
        float q2 = g[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) q2 = fmaxf(q2, g[i]);
        // (below 2^26 the roundings of the largest score and of ref are 2 each at most, and the exponent of the largest
        // probability 10 to within 4; from there on 10 would be lost in ref's)
        large = scores_may_be_large(q2, scale, 0x1p26f);
        mult = large ? 1.f : scale;
        early = large ? scale : 1.f;
        lead = large ? 0.f : 10.f;
    };
    const unsigned flip = a.scale_log2e < 0.f ? 0x80008000u : 0u;
    auto prepare_queries = [&] {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            // (the queries are waited for here, behind the first tile's requests: in the loop, they would make its
            // first product wait for the centroids of the next tile)
            u32x4 w = __builtin_bit_cast(u32x4, qreg[s]) ^ flip;
            asm volatile("" : "+v"(w));
            qreg[s] = __builtin_bit_cast(half8_t, w);
        }
    };

    if constexpr (SHORT) {
        constexpr unsigned kRaw = kRawBase(ROPE);           // the raw code tiles, one behind the other
        auto expand = [&](int k) {
            dq.request_tile_angles(a.rope_tile_tab, tile0 + k, tid);
            dq.gather(dq.kw, kRaw + (unsigned)k * kRawStageBytes, ck_head, tid, true);
            dq.gather(dq.vw, kRaw + (unsigned)k * kRawStageBytes + kTileRaw, cv_head, tid, true);
        };
        auto store = [&](int k) {
#pragma unroll
            for (int q = 0; q < D_::kRotations; ++q) dq.rotate(D_::table_angles(a.rope_lane_tab, tid, q), q);
            dq.store_keys(stage_of(tile0 + k), tid);
            dq.store_values(stage_of(tile0 + k), tid);
        };
        const int tiles = tile1 - tile0;
        if (tiles > 0) {
            constexpr int N = kShortTiles(ROPE);
            typename D_::Codes codes[N] = {};
#pragma unroll
            for (int k = 0; k < N; ++k) {
                if (k < tiles) {
                    const size_t at = a.map.tile_index(n, hkv, tile0 + k) * F::TILE_BYTES;
                    codes[k] = D_::request_codes(a.k_codes + at, a.v_codes + at, tid);
                }
            }
#pragma unroll
            for (int k = 0; k < N; ++k)
                if (k < tiles) D_::store_codes(codes[k], kRaw + (unsigned)k * kRawStageBytes, kRaw + (unsigned)k * kRawStageBytes + kTileRaw, tid);
            lds_barrier();
            expand(0);
            bound_scores();
            store(0);
        }
        prepare_queries();
        lds_barrier();
#pragma unroll 1
        for (int k = 0; k < tiles; ++k) {
            if (k + 1 < tiles) expand(k + 1);
            const unsigned stage = stage_of(tile0 + k);
            if (tile0 + k < wave_tiles) {
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[tb][i] = 0.f;
#pragma unroll
                    for (int g = tb * kGroups; g < (tb + 1) * kGroups; ++g) {
                        read_keys(stage, g);
#pragma unroll
                        for (int i = 0; i < 4; ++i) multiply_key(g, i);
                    }
                }
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) {
                    mask(tile0 + k, tb);
#pragma unroll
                    for (int q = 0; q < 10; ++q) softmax_slice(tb, q);
                    l_run = __builtin_fmaf(l_run, alpha_of[tb], psum_of[tb]);
                    rescale(tb);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        read_values(stage, tb, t);
#pragma unroll
                        for (int q = 8 * t; q < 8 * t + 8; ++q) multiply_value(tb, q);
                    }
                }
            }
            if (k + 1 < tiles) {
                store(k + 1);
                lds_barrier();
            }
        }
    } else {
        if (tile0 < tile1) {
            // (all requests first: a short context waits for them once; and of a context of one or two tiles only what it has)
            const bool two = tile0 + 1 < tile1, three = tile0 + 2 < tile1;
            const size_t first = a.map.tile_index(n, hkv, tile0);
            const typename D_::Codes c0 = D_::request_codes(a.k_codes + first * F::TILE_BYTES, a.v_codes + first * F::TILE_BYTES, tid);
            typename D_::Codes c1 = {};
            if (two) {
                const size_t second = a.map.tile_index(n, hkv, tile0 + 1);
                c1 = D_::request_codes(a.k_codes + second * F::TILE_BYTES, a.v_codes + second * F::TILE_BYTES, tid);
            }
            if (three) {
                v_index = a.map.tile_index(n, hkv, tile0 + 2);
                dq.raw = D_::request_codes(a.k_codes + v_index * F::TILE_BYTES, a.v_codes + v_index * F::TILE_BYTES, tid);
            }
            D_::store_codes(c0, k_slot(tile0), v_slot(tile0), tid);
            if (two) D_::store_codes(c1, k_slot(tile0 + 1), v_slot(tile0 + 1), tid);
            if constexpr (ROPE) {
                for (int i = tid; i < (int)kAngleBytes / 16; i += NW * 64)
                    *(lds_q*)(kAngles + (unsigned)i * 16) = reinterpret_cast<const u32x4*>(a.rope_lane_tab)[i];
            }
            dq.request_tile_angles(a.rope_tile_tab, tile0, tid);
            lds_barrier();
            dq.gather(dq.kw, k_slot(tile0), ck_head, tid, true);
            dq.gather(dq.vw, v_slot(tile0), cv_head, tid, true);
            bound_scores();
            rotate_keys();
            dq.store_keys(stage_of(tile0), tid);
            dq.store_values(stage_of(tile0), tid);
            if (two) {
                dq.gather(dq.kw, k_slot(tile0 + 1), ck_head, tid, true);
                dq.request_tile_angles(a.rope_tile_tab, tile0 + 1, tid);
            }
            if (three) {
                lds_barrier();                                  // all have read the first tile's codes
                if (tid < D_::LOADERS) *(lds_q*)(k_slot(tile0 + 2) + (unsigned)tid * 16) = dq.raw.k;
            }
        }
        prepare_queries();
        lds_barrier();

        int tile = tile0;
        for (; tile < min(tile1, wave_tiles); ++tile) {
            multiply_tile(tile);
            end_tile(tile);
        }
        // tiles behind this wavefront's rows: it still helps the others to theirs
        for (; tile < tile1; ++tile) {
            rotate_keys();
            dq.store_keys(stage_of(tile + 1), tid);
            load_codes(tile);
            dq.gather(dq.vw, v_slot(tile + 1), cv_head, tid, tile + 1 < tile1);
            dq.store_values(stage_of(tile + 1), tid);
            dq.gather(dq.kw, k_slot(tile + 2), ck_head, tid, tile + 2 < tile1);
            end_tile(tile);
        }
    }

    // ---- output: lane (rc, kh) holds channels 32 cb + 8 (i / 4) + 4 kh + i % 4 of query rc ----
    const auto lr = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
    const float l = __uint_as_float(lr[0]) + __uint_as_float(lr[1]);
    // (the row's place is formed again: held through the loop, it cost registers that spill)
    int tid_o = threadIdx.x;
    asm volatile("" : "+v"(tid_o));
    const int row_o = rb * kRowsPerWg + (tid_o >> 6) * 32 + (tid_o & 31), kh_o = tid_o >> 5 & 1;
    if (row_o >= rows_total) return;
    const int j_o = row_o / qper;
    const size_t out_row = ((size_t)n * a.m + j_o) * a.n_q_heads + hkv * qper + (row_o - j_o * qper);
    if (a.n_split == 1) {
        const float inv = 1.f / l;
        uint16_t* orow = a.out + out_row * D;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                half4_t h;
#pragma unroll
                for (int b = 0; b < 4; ++b) h[b] = (_Float16)(o[cb][4 * i4 + b] * inv);
                *reinterpret_cast<half4_t*>(orow + 32 * cb + 8 * i4 + 4 * kh_o) = h;
            }
    } else {
        float* part = a.partials + (out_row * a.n_split + split) * (D + kPartialHeader);
        if (kh_o == 0) {
            part[0] = ref;
            part[1] = l;
        }
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                float4 v;
                v.x = o[cb][4 * i4 + 0];
                v.y = o[cb][4 * i4 + 1];
                v.z = o[cb][4 * i4 + 2];
                v.w = o[cb][4 * i4 + 3];
                float* dst = part + kPartialHeader + 32 * cb + 8 * i4 + 4 * kh_o;
                dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
            }
    }
}

template <int GH, int C, int NW, int B, bool ROPE, bool SHORT>
cq_status launch_chunk_variant(const ChunkArgs& a, hipStream_t stream)
{
    auto kernel = chunk_attention_kernel<GH, C, NW, B, ROPE, SHORT>;
    static LdsKernelSetup setup;
    if (setup.ensure(reinterpret_cast<const void*>(kernel)) != hipSuccess) return CQ_ERR_HIP;
    const int qper = a.n_q_heads / a.f.n_kv_heads;
    const int row_blocks = (a.m * qper + NW * 32 - 1) / (NW * 32);
    const unsigned grid = (unsigned)(a.batch * a.n_split * row_blocks * a.f.n_kv_heads);
    const size_t lds = 2 * kStageBytes(ROPE) + (SHORT ? kShortTiles(ROPE) : 2) * Dequant<GH, C, NW, B, ROPE>::RAW_STAGE +
                       (ROPE && !SHORT ? kAngleBytes : 0);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(NW * 64), lds, stream, a);
    return hipGetLastError() == hipSuccess ? CQ_OK : CQ_ERR_HIP;
}

template <int GH, int C, int NW, int B, bool ROPE>
cq_status launch_chunk_tiles(const ChunkArgs& a, hipStream_t stream)
{
    const int n_tiles = (a.t + kTileTokens - 1) / kTileTokens;
    if ((a.tiles_per_split < n_tiles ? a.tiles_per_split : n_tiles) <= kShortTiles(ROPE)) return launch_chunk_variant<GH, C, NW, B, ROPE, true>(a, stream);
    return launch_chunk_variant<GH, C, NW, B, ROPE, false>(a, stream);
}

template <int GH, int C, int B>
cq_status launch_chunk_rows(const ChunkArgs& a, hipStream_t stream)
{
    const int rows = a.m * (a.n_q_heads / a.f.n_kv_heads);
    if (a.rope_tile_tab) {
        if (chunk_rows_per_workgroup(rows) == 128) return launch_chunk_tiles<GH, C, 4, B, true>(a, stream);
        return launch_chunk_tiles<GH, C, 8, B, true>(a, stream);
    }
    if (chunk_rows_per_workgroup(rows) == 128) return launch_chunk_tiles<GH, C, 4, B, false>(a, stream);
    return launch_chunk_tiles<GH, C, 8, B, false>(a, stream);
}

}  // namespace

int chunk_rows_per_workgroup(int rows_per_kv_head) { return rows_per_kv_head <= 128 ? 128 : 256; }

cq_status launch_chunk_attention(const ChunkArgs& a, hipStream_t stream)
{
    cq_status st = CQ_ERR_UNSUPPORTED;
    if (a.f.b == 8 && a.f.head_dim == 128) {
        if (a.f.gh == 16 && a.f.c == 8) st = launch_chunk_rows<16, 8, 8>(a, stream);
        else if (a.f.gh == 32 && a.f.c == 4) st = launch_chunk_rows<32, 4, 8>(a, stream);
        else if (a.f.gh == 64 && a.f.c == 2) st = launch_chunk_rows<64, 2, 8>(a, stream);
    } else if (a.f.b == 10 && a.f.head_dim == 128 && a.f.gh == 16 && a.f.c == 8) {
        st = launch_chunk_rows<16, 8, 10>(a, stream);
    }
    if (st != CQ_OK) return st;
    if (a.n_split > 1)
        return launch_decode_merge(a.partials, a.out, a.batch * a.m * a.n_q_heads, a.n_q_heads, (int64_t)a.n_q_heads * a.f.head_dim, a.n_split,
                                   a.f.head_dim, stream);
    return CQ_OK;
}

}  // namespace cq
