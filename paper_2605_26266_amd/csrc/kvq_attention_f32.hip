// fp32 chunk attention on the bf16 matrix cores: every cache with one (scale, zero-point) per token or group of channels,
// head_dim 64 or 128, BF16 or FP32 tensors: the caches that the 16-bit kernels do not serve, and calls with a few query rows, which
// would leave most of their 256-row blocks empty.  Queries, weights and outputs are fp32 throughout: an fp32 number enters the
// matrix instructions as three bf16 pieces that add up to it (8 + 8 + 8 significant bits), and what it is multiplied by is exact
// in bf16: key and value codes less their zero-point, times the step where that is an E4M3 number; a BF16 tensor's values.  Two
// fp32 numbers (current keys and values in fp32) take the six products above 2^-27 of the largest.  Products are exact and sums
// fp32, so the results have the precision of the vector kernel: keys scored against the rotated query, corrected by
// b = sigma^2 / 24 * sum_j step_j^2 nu_j.  What does not fit the pieces takes v_mfma_f32_32x32x2_f32 instead, tile by tile:
// zero-points that put (code - zero) beyond bf16 (fp32 pairs: beyond 240; E4M3 steps: beyond 2^20, what lies between is added
// as constants), queries and values near the ends of the fp32 range or not finite.
//
// Work split.  A unit is 32 query rows of one query head (or of the query heads that share a key/value head, one after
// the other: four heads with a row each are one unit and read the cache once); a workgroup of 8 wavefronts (two per SIMD: one unpacks while
// the other multiplies) takes a unit, or a piece of its key range, and gives each wavefront a run of its 32-key tiles.
// Each wavefront keeps its own maximum, sums and output tile; they are put together through LDS at the end, where the cached
// part is rotated back once.  Few rows (one token behind a long prefix) thereby still keep a compute unit busy, and no wavefront
// waits for another until then.  The query is rotated and cut into pieces once for the workgroup.
//
// Operands.  Everything is transposed, S^T = K Q^T and O^T = V^T P^T: a lane owns query row lane mod 32 of both result
// tiles.  The packed layout hands each lane exactly the codes it feeds to the A operand (key lane (t, hh): the channels with
// bit 3 = hh of token t; value lane (c, hh): the tokens with bit 2 = hh of channels c, c + 32, ..), so codes go from memory
// to registers to MFMA, without LDS.  Slab i of the score contracts channels 16 i .. 16 i + 15; slab sl of the output contracts
// tokens 16 sl .. 16 sl + 15 in the order in which the score leaves them in registers, so weights are B operands as they stand.
//
// Bound by instruction issue: about 420 vector instructions per tile and wave at head_dim 64 (unpacking 100, scale and softmax
// 110, weights in three pieces 104) beside 24 MFMAs.  Why this shape: with fp32 MFMAs (64 clocks for 4096 flop against 32 for
// 32768) the matrix instructions alone took 4096 (8192) clocks per tile and wave, now 768 (1536), and every wave rotated the
// query and its output by itself.  12 heads x 500 rows x (1500 + 500) keys, BF16, head_dim 64: 51.2 -> 22.4 us (137 TFLOP/s).
// 32 query heads on 8 x 1 row x (8192 + 64) keys, groups of 32: 34.4 -> 17 us (kernel alone, in 17 pieces).  4 heads x 300 rows x
// (1500 + 300) keys in fp32, head_dim 128: 39.8 -> 26.0 us (33.7 with the current tiles still on fp32 MFMAs).
#include "kvq_internal.h"

namespace kvq {
namespace {
#include "kvq_mfma_common.h"

constexpr int kFWaves = 8, kFRows = 32;
constexpr int kNotFinite = 0x207;   // class mask: either NaN, either infinity

// value of the other lane half
__device__ inline float other_half(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}
__device__ inline f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// Value of lane ^ (1, 2, 16 or 32).
template <int X> __device__ inline float lane_xor(float v)
{
    if constexpr (X == 1 || X == 2) {
        constexpr int kQuadPerm = X == 1 ? 0xb1 : 0x4e;
        return __uint_as_float(__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), kQuadPerm, 0xf, 0xf, true));
    } else if constexpr (X == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return __uint_as_float((threadIdx.x & 16) ? r[0] : r[1]);
    } else {
        return other_half(v);
    }
}

// fp32 pairs as three bf16 pairs that add up to them (8 + 8 + 8 significant bits)
struct Pieces {
    uint32_t hi, mid, lo;
};
__device__ inline float lower(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float upper(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ inline Pieces split3(float x, float y)
{
    Pieces p;
    p.hi = pack_bf16(x, y);
    x -= lower(p.hi); y -= upper(p.hi);
    p.mid = pack_bf16(x, y);
    x -= lower(p.mid); y -= upper(p.mid);
    p.lo = pack_bf16(x, y);
    return p;
}
typedef __attribute__((ext_vector_type(4))) short i16x4;
__device__ inline u32x2 read_transposed(const uint16_t *p)
{
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)p));
}
// Products of two numbers in three pieces each, less what lies 27 bits and more below the largest
__device__ inline f32x16 mfma_pieces(const u32x4 (&x)[3], const u32x4 (&y)[3], f32x16 c)
{
    c = mfma_bf16(x[2], y[0], c);
    c = mfma_bf16(x[1], y[1], c);
    c = mfma_bf16(x[0], y[2], c);
    c = mfma_bf16(x[1], y[0], c);
    c = mfma_bf16(x[0], y[1], c);
    return mfma_bf16(x[0], y[0], c);
}
// Four codes of a word, one per byte: pairs J and J + 4 (2-bit codes) or J + 2 (4-bit codes) in bytes 0, 2 and 1, 3.
template <int BITS> __device__ inline uint32_t four_codes(uint32_t w, int j)
{
    uint32_t t = (w >> (BITS * j)) & (BITS == 2 ? 0x03030303u : 0x0f0f0f0fu);
    asm("" : "+v"(t));       // (one conversion per byte, not a bit field extraction before each)
    return t;
}
__device__ inline float byte0(uint32_t t) { return (float)(t & 0xffu); }
__device__ inline float byte1(uint32_t t) { return (float)((t >> 8) & 0xffu); }
__device__ inline float byte2(uint32_t t) { return (float)((t >> 16) & 0xffu); }
__device__ inline float byte3(uint32_t t) { return (float)(t >> 24); }
// The bf16 values of four codes from tables of their low and high bytes: pairs from bytes 0, 2 and 1, 3.
__device__ inline void look_up(uint32_t t, uint32_t low, uint32_t high, uint32_t &even, uint32_t &odd)
{
    const uint32_t l = __builtin_amdgcn_perm(0u, low, t), h = __builtin_amdgcn_perm(0u, high, t);
    even = __builtin_amdgcn_perm(h, l, 0x06020400u);
    odd = __builtin_amdgcn_perm(h, l, 0x07030501u);
}
__device__ inline void set(u32x4 &q, int i, uint32_t w)
{
    if (i == 0) q.x = w;
    else if (i == 1) q.y = w;
    else if (i == 2) q.z = w;
    else q.w = w;
}

// 8 consecutive channels
__device__ inline void load8(const float *p, float (&x)[8])
{
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}
__device__ inline void load8(const uint16_t *p, float (&x)[8])
{
    const u32x4 w = *reinterpret_cast<const u32x4 *>(p);
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        x[2 * j] = __uint_as_float(ws[j] << 16);
        x[2 * j + 1] = __uint_as_float(ws[j] & 0xffff0000u);
    }
}
// E4M3 scales and BF16 zero-points of a token's G groups
template <int G> __device__ inline void load_scales(const uint8_t *p, float (&x)[G])
{
    const uint32_t w = G == 4 ? *reinterpret_cast<const uint32_t *>(p) : G == 2 ? *reinterpret_cast<const uint16_t *>(p) : *p;
    x[0] = __builtin_amdgcn_cvt_f32_fp8((int)w, 0);
    if constexpr (G > 1) x[1] = __builtin_amdgcn_cvt_f32_fp8((int)w, 1);
    if constexpr (G > 2) {
        x[2] = __builtin_amdgcn_cvt_f32_fp8((int)w, 2);
        x[3] = __builtin_amdgcn_cvt_f32_fp8((int)w, 3);
    }
}
template <int G> __device__ inline void load_zeros(const uint16_t *p, float (&x)[G])
{
    if constexpr (G == 1) {
        x[0] = bf16_to_float(*p);
    } else {
#pragma unroll
        for (int j = 0; j < G; j += 2) {
            const uint32_t w = reinterpret_cast<const uint32_t *>(p)[j >> 1];
            x[j] = lower(w);
            x[j + 1] = upper(w);
        }
    }
}
__device__ inline void store4(float *p, float a, float b, float c, float d) { *reinterpret_cast<float4 *>(p) = float4{a, b, c, d}; }
__device__ inline void store4(uint16_t *p, float a, float b, float c, float d)
{
    *reinterpret_cast<uint2 *>(p) = uint2{(uint32_t)float_to_bf16(a) | ((uint32_t)float_to_bf16(b) << 16),
                                          (uint32_t)float_to_bf16(c) | ((uint32_t)float_to_bf16(d) << 16)};
}

// LDS, in words.  While tiles are worked on: query pieces [piece][slab][lane][4], the query in fp32 [slab][quad][lane][4], fp32 tensors: pieces of
// the query before rotation; correction factors and, once asked for, the query's sums over groups [group][row], metadata
// of each wave's tile [value scale | value zero | key scale, or what the value zero-points leave | what the key ones leave][group][token], and for each wave the weights or the values of a tile; later the waves' outputs; behind both the
// waves' maxima and sums.
template <int DIM, int G, bool BF16> struct F32Lds {
    static constexpr int kPieces = 3 * (DIM / 16) * 256, kQuery = kPieces, kPlain = kQuery + DIM * 32, kCorr = kPlain + (BF16 ? 0 : kPieces), kSum = kCorr + G * 32, kMeta = kSum + G * 32, kMetaWave = 4 * G * 32;
    static constexpr int kFlags = kMeta + kFWaves * kMetaWave, kOwn = kFlags + kFWaves;
    // BF16 value rows of a current tile, 64 bytes longer than the row (four rows and two 16-channel columns fill the banks once)
    static constexpr int kStageRow = DIM + 32, kStageWave = kTileTokens * kStageRow / 2;
    // A wave's own area holds its weights or its values: waves need not be at the same kind of tile.
    static constexpr int kWeightsWave = 16 * 64, kOwnWave = BF16 && kStageWave > kWeightsWave ? kStageWave : kWeightsWave;
    static constexpr int kWork = kOwn + kFWaves * kOwnWave;
    static_assert(kOwnWave >= kWeightsWave && (!BF16 || kOwnWave >= kStageWave), "neither reaches into the next wave's area");
    static_assert(kOwn % 4 == 0 && kOwnWave % 4 == 0, "16-byte accesses");
    // Outputs: [register quad][lane][4], the quads 16 words apart so that the threads that add the waves' up find their channels
    // in different banks.  A wave that has cached and current tiles leaves two of them, the first while others still work.
    static constexpr int kQuad = 256 + 16, kSlot = DIM / 8 * kQuad, kOut = kFWaves * kSlot;
    static constexpr int kSlot8 = kWork > kOut ? kWork : kOut;
    static constexpr int kRed = kSlot8 + kSlot, kWords = kRed + (kFWaves + 1) * 32 * 4;
};

// GROUP: channels per (scale, zero-point); DIM and fp32 pairs for KVQ_META_FP32, FP8: E4M3 / BF16 encodings.
template <int DIM, int BITS, typename T, bool FP8, int GROUP>
__global__ __launch_bounds__(64 * kFWaves, 2) void attention_f32_kernel(AttentionArgs a, SplitArgs sp)
{
    constexpr int WPL = DIM * BITS / 64;          // words of a lane's codes per tile
    constexpr int NI = DIM / 16, NB = DIM / 32;   // channel slabs of the score, channel blocks of the output
    constexpr int G = DIM / GROUP;
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    constexpr float kNorm = DIM == 64 ? 0.125f : 0.088388347648318f;
    constexpr bool kBf16 = sizeof(T) == 2;
    using L = F32Lds<DIM, G, kBf16>;
    extern __shared__ __align__(16) float lds[];
    const CacheView &cv = a.cv;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 31, hh = lane >> 5;

    // unit and piece
    int unit, split = 0, piece = -1;
    if ((int)blockIdx.x < sp.whole) {
        unit = xcd_contiguous(blockIdx.x, sp.whole);
    } else {
        piece = xcd_contiguous((int)blockIdx.x - sp.whole, sp.pieces);
        unit = sp.whole + piece / sp.splits;
        split = piece % sp.splits;
    }
    // Rows of the query heads that share a key/value head follow one another where `pack` says so.
    const int rblk = unit % sp.row_blocks, qhead0 = unit / sp.row_blocks * sp.pack, head = qhead0 / a.q_per_kv;
    const int64_t rows = a.m * sp.pack, block_row0 = (int64_t)rblk * kFRows;
    // row of the call and query head of row r of the block (the last row again past the end)
    auto find_row = [&](int r, int64_t &row, int &qhead) {
        const int64_t packed_row = block_row0 + r < rows ? block_row0 + r : rows - 1;
        qhead = qhead0;
        row = packed_row;
        if (sp.pack > 1) {
            qhead += (int)((uint32_t)packed_row / (uint32_t)a.m);
            row = (uint32_t)packed_row % (uint32_t)a.m;
        }
    };
    int64_t row;
    int qhead;
    find_row(n, row, qhead);
    // current keys this row sees, and some row of the block
    int64_t visible = a.n_cur, n_keys = a.n_cur;
    if (a.causal) {
        // the last row of the block, or of a head that ends inside it
        const int64_t end = block_row0 + kFRows < rows ? block_row0 + kFRows : rows;
        int64_t last = end - 1;
        if (sp.pack > 1) last = (uint32_t)block_row0 / (uint32_t)a.m != (uint32_t)(end - 1) / (uint32_t)a.m ? a.m - 1 : (uint32_t)(end - 1) % (uint32_t)a.m;
        const int64_t upto = row + (a.n_cur - a.m) + 1, upto_last = last + (a.n_cur - a.m) + 1;
        visible = upto < visible ? upto : visible;
        n_keys = upto_last < n_keys ? upto_last : n_keys;
    }
    const int64_t t_first = a.cache_start / kTileTokens;
    const int tc = a.cache_len > 0 ? (int)((a.cache_start + a.cache_len - 1) / kTileTokens - t_first) + 1 : 0;
    const int all = tc + (int)((n_keys + kTileTokens - 1) / kTileTokens);
    int x0 = 0, x1 = all;
    if (piece >= 0) {          // all * split / splits and all * (split + 1) / splits, without their 64-bit products
        const int each = all / sp.splits, left = all - each * sp.splits;
        x0 = each * split + left * split / sp.splits;
        x1 = each * (split + 1) + left * (split + 1) / sp.splits;
    }
    const int first_off = (int)(a.cache_start - t_first * kTileTokens);

    const float c_log = a.softmax_scale * kLog2e;
    const T *const q_all = static_cast<const T *>(a.q);

    // weights of a tile in LDS, for loops that cannot index registers
    float *const weights = lds + L::kOwn + wave * L::kOwnWave;
    auto keep_weights = [&](const f32x16 &s) {
#pragma unroll
        for (int v = 0; v < 16; ++v) weights[64 * v + lane] = s[v];
    };

    // Eight consecutive channels of a row for each thread: lane bits 0, 1, 4 (and 5 for head_dim 128) are bits 3, 4, 5 (6) of the
    // channel, so the butterflies across lanes need no LDS.
    constexpr int kGroups = DIM / 8;
    const bool has_octet = kGroups == 16 || wave < 4;
    const int g8 = (lane & 3) | ((lane >> 2) & 4) | (kGroups == 16 ? (lane >> 2) & 8 : 0);
    const int r8 = ((lane >> 2) & 3) | (kGroups == 16 ? wave << 2 : ((lane >> 3) & 4) | ((wave & 3) << 3));
    int64_t row8;
    int qhead8;
    find_row(r8, row8, qhead8);
    auto hadamard = [&](float (&y)[8]) {
#pragma unroll
        for (int h = 1; h < 8; h <<= 1)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if ((e & h) == 0) {
                    const float p = y[e], q = y[e + h];
                    y[e] = p + q;
                    y[e + h] = p - q;
                }
        auto across = [&](auto xor_lanes) {
            constexpr int X = decltype(xor_lanes)::value;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float q = lane_xor<X>(y[e]);
                y[e] = lane & X ? q - y[e] : y[e] + q;
            }
        };
        across(IntC<1>{});
        across(IntC<2>{});
        across(IntC<16>{});
        if constexpr (kGroups == 16) across(IntC<32>{});
    };

    // ---- this wave's tiles: a run of them, so that one wave at most has cached and current tiles.  The first cached one is requested
    // before the query is prepared.
    const int each = (x1 - x0) / kFWaves, left = (x1 - x0) % kFWaves;
    auto run_start = [&](int w) { return x0 + w * each + (w < left ? w : left); };
    int x = run_start(wave);
    const int x_end = run_start(wave + 1), c_end = x_end < tc ? x_end : tc;
    const int64_t cap = cv.cap_tiles, head_tile0 = (int64_t)head * cap;
    const float off = code_offset(BITS);
    uint32_t kw[WPL], vw[WPL];
    float ks[G], kz[G], vs[G], vz[G];
    bool seen;
    auto tile_token = [&](int tile) {                   // place of the tile's first token in the storage
        int64_t phys = a.phys_tile_first + tile;        // a window has at most cap + 1 tiles
        phys -= phys >= cap ? cap : 0;
        phys -= phys >= cap ? cap : 0;
        return (head_tile0 + phys) * kTileTokens;
    };
    auto fetch = [&](int tile) {
        const int64_t tok = tile_token(tile) + n, word = (tile_token(tile) / kTileTokens * 64 + lane) * WPL;
        if constexpr (WPL >= 4) {
#pragma unroll
            for (int i = 0; i < WPL; i += 4) {
                const u32x4 k4 = *reinterpret_cast<const u32x4 *>(cv.k_codes + word + i), v4 = *reinterpret_cast<const u32x4 *>(cv.v_codes + word + i);
                kw[i] = k4.x; kw[i + 1] = k4.y; kw[i + 2] = k4.z; kw[i + 3] = k4.w;
                vw[i] = v4.x; vw[i + 1] = v4.y; vw[i + 2] = v4.z; vw[i + 3] = v4.w;
            }
        } else {
            const u32x2 k2 = *reinterpret_cast<const u32x2 *>(cv.k_codes + word), v2 = *reinterpret_cast<const u32x2 *>(cv.v_codes + word);
            kw[0] = k2.x; kw[1] = k2.y;
            vw[0] = v2.x; vw[1] = v2.y;
        }
        // Tokens outside the window keep nothing of what the storage holds there: step and zero-point 0.
        const int rel = tile * kTileTokens + n - first_off;
        seen = rel >= 0 && rel < a.cache_len;
        if constexpr (FP8) {           // (a token's groups lie side by side, aligned to their size)
            load_scales<G>(cv.k_scale8 + tok * G, ks);
            load_scales<G>(cv.v_scale8 + tok * G, vs);
            load_zeros<G>(cv.k_zero16 + tok * G, kz);
            load_zeros<G>(cv.v_zero16 + tok * G, vz);
        } else {
            ks[0] = cv.k_scale[tok];
            vs[0] = cv.v_scale[tok];
            kz[0] = -cv.k_negzero[tok] - off;
            vz[0] = cv.v_zero_off[tok] - off;
        }
    };
    if (x < c_end) fetch(x);

    // ---- query in pieces, once for the eight waves: rotated for the cached keys, as it is for current ones in fp32
    uint32_t *const pieces = reinterpret_cast<uint32_t *>(lds);
    // Operands so small that their third pieces may be lost, so large that sums of pieces may overflow, or not finite: fp32 products.
    // Queries and current keys meet each other: below 2^63 each, where no product of pieces overflows that the score itself does not
    // (high times middle piece may be +inf beside -inf of the high ones).
    constexpr float kTop = 0x1p100f, kTopFactor = 0x1p63f;
    auto in_range = [](float sum, float top) { return sum == 0.0f || (sum >= 0x1p-90f && sum <= top); };
    bool unfit = false;
    if (x0 < tc || !kBf16) {               // (the same for all waves)
        if (has_octet) {
            float y[8];
            auto leave_pieces = [&](uint32_t *dst) {
                u32x4 piece[3];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const Pieces s = split3(y[2 * p], y[2 * p + 1]);
                    set(piece[0], p, s.hi);
                    set(piece[1], p, s.mid);
                    set(piece[2], p, s.lo);
                }
#pragma unroll
                for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4 *>(dst + 4 * ((p * NI + (g8 >> 1)) * 64 + 32 * (g8 & 1) + r8)) = piece[p];
            };
            load8(q_all + row8 * a.q_stride_token + (int64_t)qhead8 * a.q_stride_head + 8 * g8, y);
            if constexpr (!kBf16) {
                float x8[8], sum = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    x8[e] = y[e];
                    y[e] *= c_log;
                    sum += fabsf(y[e]);
                }
                unfit = !in_range(sum, kTopFactor);
                leave_pieces(pieces + L::kPlain);
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = x8[e];
            }
            if (has_signs(cv)) {
                const uint32_t sg = sign_bits_from(cv, 8 * g8);
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = flip_sign(y[e], (sg >> e) & 1u);
            }
            hadamard(y);
            float nu = 0.0f, sum = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                y[e] *= kNorm;
                nu = fmaf(y[e], y[e], nu);
                y[e] *= c_log;
                sum += fabsf(y[e]);
            }
            nu += lane_xor<1>(nu);
            nu += lane_xor<2>(nu);
            if constexpr (GROUP >= 64) nu += lane_xor<16>(nu);
            if constexpr (GROUP >= 128) nu += lane_xor<32>(nu);
            if (g8 % (GROUP / 8) == 0)
                lds[L::kCorr + g8 / (GROUP / 8) * 32 + r8] = a.correction == 1 ? -nu * (a.softmax_scale * c_log * (1.0f / 24.0f)) : 0.0f;
            leave_pieces(pieces);
#pragma unroll
            for (int p = 0; p < 2; ++p)
                *reinterpret_cast<float4 *>(lds + L::kQuery + 4 * (((g8 >> 1) * 2 + p) * 64 + 32 * (g8 & 1) + r8)) =
                    float4{y[4 * p], y[4 * p + 1], y[4 * p + 2], y[4 * p + 3]};
            unfit = unfit || !in_range(sum, kTop);
        }
        const bool any_unfit = __any(unfit);
        if (lane == 0) pieces[L::kFlags + wave] = any_unfit;
        __syncthreads();
        uint32_t flags = 0;
#pragma unroll
        for (int w = 0; w < kFWaves; ++w) flags |= pieces[L::kFlags + w];
        unfit = __builtin_amdgcn_readfirstlane(flags) != 0u;
    }

    f32x16 o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[b][v] = 0.0f;
    // Scores are taken relative to `base`, which moves when a row goes beyond it by more than a factor of 2^slack (weights and sums
    // are fp32: where it lies matters only to sums that come near the end of the range).  `above`: the row's largest score less
    // `base`, -inf before the first one.
    float base = 0.0f, above = -INFINITY, slack = 8.0f, l_s = 0.0f, l_r = 0.0f, tau = 0.0f;

    // s: scores in log2 units less `base` (-inf: key not seen) -> weights.  large: the tile's values lie so high that sums with
    // weights up to 2^slack might leave the range of fp32; from here on weights stay below 1.
    auto weigh = [&](f32x16 &s, float &l, bool large) {
        if (__builtin_expect(large, 0)) slack = 0.0f;
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        mx = fmaxf(mx, other_half(mx));
        const bool first = above == -INFINITY;
        above = fmaxf(above, mx);
        const bool moves = above > (first ? -INFINITY : slack);
        if (__any(moves)) {
            const float to = moves ? base + above : base, by = to - base, alpha = first ? 1.0f : __builtin_amdgcn_exp2f(-by);
            base = to;
            above = moves ? 0.0f : above;
            l_s *= alpha;
            l_r *= alpha;
            tau *= alpha;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[b][v] *= alpha;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] -= by;
        }
        float sum = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(s[v]);
            sum += s[v];
        }
        l += sum;
    };

    // ---- cached tiles
    if (x < c_end) {
        constexpr int kKept = DIM == 64 ? 3 : 1;      // pieces of the query in registers; the others are read for every tile
        u32x4 qp[kKept][NI];
        const uint32_t *const my_pieces = pieces + 4 * lane;
#pragma unroll
        for (int p = 0; p < kKept; ++p)
#pragma unroll
            for (int i = 0; i < NI; ++i) qp[p][i] = *reinterpret_cast<const u32x4 *>(my_pieces + 256 * (p * NI + i));
        auto query = [&](int p, int i) { return p < kKept ? qp[p % kKept][i] : *reinterpret_cast<const u32x4 *>(my_pieces + 256 * (p * NI + i)); };
        constexpr bool kTau = !FP8 && BITS == 2;
        float corr[G];
#pragma unroll
        for (int j = 0; j < G; ++j) corr[j] = lds[L::kCorr + j * 32 + n];
        // correction as an operand: squared E4M3 steps are bf16 values, the factors are taken in three pieces (groups 2 hh, 2 hh + 1)
        u32x4 corr_op = {0u, 0u, 0u, 0u};
        if constexpr (FP8) {
            const float c0 = G == 4 ? (hh ? corr[2 % G] : corr[0]) : hh ? (G == 2 ? corr[1 % G] : 0.0f) : corr[0];
            const float c1 = G == 4 ? (hh ? corr[3 % G] : corr[1 % G]) : 0.0f;
            const Pieces s = split3(c0, c1);
            corr_op.x = (s.hi & 0xffffu) | (s.mid << 16);
            corr_op.y = (s.lo & 0xffffu) | (s.hi & 0xffff0000u);
            corr_op.z = (s.mid >> 16) | (s.lo & 0xffff0000u);
        }
        float *const meta = lds + L::kMeta + wave * L::kMetaWave;      // this wave's metadata: [value scale | zero | key scale][group][token]
        // Register v of a result tile holds key (token) 8 (v >> 2) + 4 hh + (v & 3).
        auto per_key = [&](int row, int g4) { return *reinterpret_cast<const float4 *>(meta + row * 32 + 8 * g4 + 4 * hh); };
        bool have_sums = false;
        for (;;) {
            const int tile = x;
            const bool edge = tile == 0 || tile == tc - 1;
            if (!seen) {
#pragma unroll
                for (int j = 0; j < G; ++j) ks[j] = kz[j] = vs[j] = vz[j] = 0.0f;
            }
            // What the 16-bit operands hold exactly: (code - zero) up to 256; times a step of four significant bits, up to 15.
            // (kTau: values are code - 1, the middle of their range, and what is left of the zero-points goes into tau.)
            // Steps whose products with weights may leave the range at either end are not among them.
            constexpr float kMid = FP8 ? 0.5f * (float)MASK : 0.0f, kFar = FP8 ? 15.0f - 0.5f * (float)MASK : 240.0f;
            bool fits_k = !unfit, fits_v = FP8 || vs[0] == 0.0f || (vs[0] >= 0x1p-80f && vs[0] <= 0x1p80f);
            if (kTau) fits_v = fits_v && fabsf(vz[0]) * vs[0] <= kTop;
#pragma unroll
            for (int j = 0; j < G; ++j) {
                fits_k = fits_k && fabsf(kz[j] - kMid) <= kFar;
                if (!kTau) fits_v = fits_v && fabsf(vz[j] - kMid) <= kFar;
            }
            fits_k = __all(fits_k);
            fits_v = __all(fits_v);
            // E4M3 steps: every group of 4-bit codes whose range does not hold 0 has a zero-point beyond 0 .. 15.  The operand takes
            // the nearest one within, and what that leaves, the same for all channels of the group, is added as a constant of the
            // key (times the query's sum over the group) or of the value (on all channels of the group).  As fp32 MFMAs such tiles
            // took twice the time and more (12 heads x 500 rows x (1500 + 500) keys, head_dim 64, BF16, 4 bits, groups of 32: 26 us on
            // centred values; with one large key channel and an offset of the values 66 us that way, 29 this way).  Work that such tiles alone need stands at
            // branches that were there: sums over the query in its preparation and a branch inside the scores cost every call 0.4 us.
            constexpr float kLow = (float)MASK - 15.0f, kHigh = 15.0f, kExact = 0x1p20f;
            bool far_k = false, far_v = false;
            if constexpr (FP8) {
                far_k = !fits_k && !unfit;
                far_v = !fits_v;
                if (__builtin_expect(far_k || far_v, 0)) {
                    fits_k = !unfit;
                    fits_v = true;
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        fits_k = fits_k && fabsf(kz[j]) <= kExact;
                        fits_v = fits_v && fabsf(vz[j]) <= kExact;
                    }
                    fits_k = __all(fits_k);
                    fits_v = __all(fits_v);
                    far_k = far_k && fits_k;
                    far_v = far_v && fits_v;
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        const float k = far_k ? __builtin_amdgcn_fmed3f(kz[j], kLow, kHigh) : kz[j];
                        const float v = far_v ? __builtin_amdgcn_fmed3f(vz[j], kLow, kHigh) : vz[j];
                        meta[((2 + hh) * G + j) * 32 + n] = hh ? (k - kz[j]) * ks[j] : (v - vz[j]) * vs[j];
                        kz[j] = k;
                        vz[j] = v;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < G; ++j) {
                meta[(hh * G + j) * 32 + n] = hh ? (!fits_v ? -vz[j] : FP8 ? -vz[j] * vs[j] : kTau ? 1.0f - vz[j] : -vz[j]) : vs[j];
                if (!FP8 && hh == 0) meta[(2 * G + j) * 32 + n] = ks[j];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            f32x16 s;
            if (__builtin_expect(fits_k, 1)) {
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = 0.0f;
                if constexpr (FP8) {
                    const float s0 = G == 4 ? (hh ? ks[2 % G] : ks[0]) : hh ? (G == 2 ? ks[1 % G] : 0.0f) : ks[0];
                    const float s1 = G == 4 ? (hh ? ks[3 % G] : ks[1 % G]) : 0.0f;
                    const uint32_t w = pack_bf16(s0 * s0, s1 * s1);
                    const uint32_t w0 = (w & 0xffffu) * 0x10001u, w1 = (w >> 16) * 0x10001u;
                    s = mfma_bf16(u32x4{w0, (w0 & 0xffffu) | (w1 & 0xffff0000u), w1, 0u}, corr_op, s);
                }
                auto multiply = [&](const u32x4 &op, int i) {
                    s = mfma_bf16(op, query(2, i), s);
                    s = mfma_bf16(op, query(1, i), s);
                    s = mfma_bf16(op, query(0, i), s);
                };
                if constexpr (BITS == 2) {
                    uint32_t low = 0, high = 0;
#pragma unroll
                    for (int i = 0; i < NI; i += 2) {
                        const int j = 16 * i / GROUP;
                        if (16 * i % GROUP == 0) {      // the four values of a code
                            const float st = FP8 ? ks[j] : 1.0f, add = FP8 ? -kz[j] * ks[j] : -kz[j];
                            const uint32_t e01 = __builtin_amdgcn_perm(__float_as_uint(st + add), __float_as_uint(add), 0x07060302u);
                            const uint32_t e23 = __builtin_amdgcn_perm(__float_as_uint(fmaf(3.0f, st, add)), __float_as_uint(fmaf(2.0f, st, add)), 0x07060302u);
                            low = __builtin_amdgcn_perm(e23, e01, 0x06040200u);
                            high = __builtin_amdgcn_perm(e23, e01, 0x07050301u);
                        }
                        u32x4 op0, op1;
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            uint32_t even, odd;
                            look_up(four_codes<BITS>(kw[i >> 1], p), low, high, even, odd);
                            set(op0, p, even);
                            set(op1, p, odd);
                        }
                        multiply(op0, i);
                        multiply(op1, i + 1);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        const int j = 16 * i / GROUP;
                        const float st = FP8 ? ks[j] : 1.0f, add = FP8 ? -kz[j] * ks[j] : -kz[j];
                        u32x4 op;
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            const uint32_t t = four_codes<BITS>(kw[i % WPL], p);
                            set(op, p, pack_bf16(fmaf(byte0(t), st, add), fmaf(byte2(t), st, add)));
                            set(op, p + 2, pack_bf16(fmaf(byte1(t), st, add), fmaf(byte3(t), st, add)));
                        }
                        multiply(op, i);
                    }
                }
                if constexpr (FP8) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) s[v] -= base;
                } else {
#pragma unroll
                    for (int g4 = 0; g4 < 4; ++g4) {
                        const float4 k4 = per_key(2, g4);
                        const float k[4] = {k4.x, k4.y, k4.z, k4.w};
#pragma unroll
                        for (int r = 0; r < 4; ++r) s[4 * g4 + r] = fmaf(k[r], fmaf(corr[0], k[r], s[4 * g4 + r]), -base);
                    }
                }
            } else {
                // (rolled up, with everything read again: rarely run, and the registers belong to the path above)
                const int64_t tok = tile_token(tile) + n;
                const uint32_t *const words = cv.k_codes + (tile_token(tile) / kTileTokens * 64 + lane) * WPL;
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = 0.0f;
                // The square of an fp32 step can overflow where the correction is ordinary: factor by factor.
                if constexpr (!FP8) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float st = meta[2 * 32 + 8 * (v >> 2) + 4 * hh + (v & 3)];
                        s[v] = corr[0] * st * st;
                    }
                } else {
#pragma unroll 1
                    for (int j = 0; j < G; ++j) {
                        const float st = seen && hh == 0 ? e4m3_low_byte(cv.k_scale8[tok * G + j]) : 0.0f;
                        s = mfma_f32(st * st, lds[L::kCorr + j * 32 + n], s);
                    }
                }
#pragma unroll 1
                for (int i = 0; i < NI; ++i) {
                    const uint32_t w = BITS == 2 ? words[i >> 1] >> (8 * (i & 1)) : words[i];
                    const int j = 16 * i / GROUP;
                    float scale = 0.0f, zero = 0.0f;
                    if (seen) {
                        scale = FP8 ? e4m3_low_byte(cv.k_scale8[tok * G + j]) : ks[0];
                        zero = FP8 ? bf16_to_float(cv.k_zero16[tok * G + j]) : kz[0];
                    }
                    const float4 q0 = *reinterpret_cast<const float4 *>(lds + L::kQuery + 4 * (2 * i * 64 + lane));
                    const float4 q1 = *reinterpret_cast<const float4 *>(lds + L::kQuery + 4 * ((2 * i + 1) * 64 + lane));
                    const float q[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float code = (float)((w >> (BITS * (e >> 1) + 16 * (e & 1))) & MASK);
                        s = mfma_f32((code - zero) * scale, q[e], s);
                    }
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] -= base;
            }
            uint32_t vcur[WPL];
#pragma unroll
            for (int i = 0; i < WPL; ++i) vcur[i] = vw[i];
            const bool more = ++x < c_end;
            if (more) fetch(x);
            if (FP8 && __builtin_expect(far_k, 0)) {
                // what is left of the zero-points times the query's sum over the group: both factors in three pieces, the six
                // products above 2^-27 (lane half hh: group g + hh)
                if (!have_sums) {       // (waves that come here write the same sums to the same place)
                    have_sums = true;
#pragma unroll 1
                    for (int g = 0; g < G; ++g) {
                        float sum = 0.0f;
#pragma unroll 1
                        for (int i = g * (GROUP / 8); i < (g + 1) * (GROUP / 8); ++i) {      // quads of this lane half's channels
                            const float4 x = *reinterpret_cast<const float4 *>(lds + L::kQuery + 4 * (i * 64 + lane));
                            sum += (x.x + x.y) + (x.z + x.w);
                        }
                        lds[L::kSum + g * 32 + n] = sum + other_half(sum);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
#pragma unroll
                for (int g = 0; g < G; g += 2) {
                    const float rest = G == 1 && hh ? 0.0f : meta[(3 * G + (G == 1 ? 0 : g + hh)) * 32 + n];
                    const float q_sum = lds[L::kSum + (G == 1 ? 0 : g + hh) * 32 + n];
                    const Pieces e = split3(rest, rest), q = split3(q_sum, q_sum);
                    constexpr uint32_t kLowHalf = 0xffffu, kHighHalf = 0xffff0000u;
                    s = mfma_bf16(u32x4{(e.hi & kLowHalf) | (e.mid & kHighHalf), (e.lo & kLowHalf) | (e.mid & kHighHalf), e.hi, 0u},
                                  u32x4{(q.lo & kLowHalf) | (q.mid & kHighHalf), q.hi, (q.mid & kLowHalf) | (q.hi & kHighHalf), 0u}, s);
                }
            }
            if (edge) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int rel = tile * kTileTokens + 8 * (v >> 2) + 4 * hh + (v & 3) - first_off;
                    s[v] = rel >= 0 && rel < a.cache_len ? s[v] : -INFINITY;
                }
            }
            weigh(s, l_s, !fits_v);
            if (__builtin_expect(fits_v, 1)) {
                if (FP8 && __builtin_expect(far_v, 0)) {
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        float t = 0.0f;
#pragma unroll
                        for (int g4 = 0; g4 < 4; ++g4) {
                            const float4 e = per_key(2 * G + j, g4);
                            t = fmaf(s[4 * g4], e.x, t); t = fmaf(s[4 * g4 + 1], e.y, t); t = fmaf(s[4 * g4 + 2], e.z, t); t = fmaf(s[4 * g4 + 3], e.w, t);
                        }
                        t += other_half(t);
#pragma unroll
                        for (int b = 0; b < GROUP / 32; ++b)
#pragma unroll
                            for (int v = 0; v < 16; ++v) o[j * (GROUP / 32) + b][v] += t;
                    }
                }
                if constexpr (!FP8) {
#pragma unroll
                    for (int g4 = 0; g4 < 4; ++g4) {
                        const float4 v4 = per_key(0, g4), z4 = per_key(1, g4);
                        const float sc[4] = {v4.x, v4.y, v4.z, v4.w}, nz[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            s[4 * g4 + r] *= sc[r];
                            if constexpr (kTau) tau = fmaf(s[4 * g4 + r], nz[r], tau);
                        }
                    }
                }
                u32x4 pp[3][2];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const Pieces t = split3(s[2 * i], s[2 * i + 1]);
                    set(pp[0][i >> 2], i & 3, t.hi);
                    set(pp[1][i >> 2], i & 3, t.mid);
                    set(pp[2][i >> 2], i & 3, t.lo);
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int j = 32 * b / GROUP;
                    u32x4 op[2];
                    // pair p of token slab sl: tokens 16 sl + 8 (p >> 1) + 4 hh + 2 (p & 1), + 1
                    if constexpr (BITS == 2) {
#pragma unroll
                        for (int p2 = 0; p2 < 2; ++p2) {
                            const float4 s0 = FP8 ? per_key(j, p2) : float4{}, a0 = FP8 ? per_key(G + j, p2) : float4{};
                            const float4 s1 = FP8 ? per_key(j, 2 + p2) : float4{}, a1 = FP8 ? per_key(G + j, 2 + p2) : float4{};
#pragma unroll
                            for (int e = 0; e < 2; ++e) {
                                const uint32_t t = four_codes<BITS>(vcur[b % WPL], 2 * p2 + e);
                                uint32_t even, odd;
                                if constexpr (FP8) {
                                    even = e ? pack_bf16(fmaf(byte0(t), s0.z, a0.z), fmaf(byte2(t), s0.w, a0.w))
                                             : pack_bf16(fmaf(byte0(t), s0.x, a0.x), fmaf(byte2(t), s0.y, a0.y));
                                    odd = e ? pack_bf16(fmaf(byte1(t), s1.z, a1.z), fmaf(byte3(t), s1.w, a1.w))
                                            : pack_bf16(fmaf(byte1(t), s1.x, a1.x), fmaf(byte3(t), s1.y, a1.y));
                                } else {
                                    look_up(t, 0x00800080u, 0x403f00bfu, even, odd);      // -1, 0, 1, 2
                                }
                                set(op[0], 2 * p2 + e, even);
                                set(op[1], 2 * p2 + e, odd);
                            }
                        }
                    } else {
#pragma unroll
                        for (int sl = 0; sl < 2; ++sl) {
                            const float4 one = {1.0f, 1.0f, 1.0f, 1.0f};
                            const float4 s0 = FP8 ? per_key(j, 2 * sl) : one, a0 = per_key(G + j, 2 * sl);
                            const float4 s1 = FP8 ? per_key(j, 2 * sl + 1) : one, a1 = per_key(G + j, 2 * sl + 1);
#pragma unroll
                            for (int p = 0; p < 2; ++p) {
                                const uint32_t t = four_codes<BITS>(vcur[(2 * b + sl) % WPL], p);
                                const uint32_t first = p ? pack_bf16(fmaf(byte0(t), s0.z, a0.z), fmaf(byte2(t), s0.w, a0.w))
                                                         : pack_bf16(fmaf(byte0(t), s0.x, a0.x), fmaf(byte2(t), s0.y, a0.y));
                                const uint32_t second = p ? pack_bf16(fmaf(byte1(t), s1.z, a1.z), fmaf(byte3(t), s1.w, a1.w))
                                                          : pack_bf16(fmaf(byte1(t), s1.x, a1.x), fmaf(byte3(t), s1.y, a1.y));
                                set(op[sl], p, first);
                                set(op[sl], p + 2, second);
                            }
                        }
                    }
#pragma unroll
                    for (int sl = 0; sl < 2; ++sl)
#pragma unroll
                        for (int p = 2; p >= 0; --p) o[b] = mfma_bf16(op[sl], pp[p][sl], o[b]);
                }
            } else {
                const uint32_t *const words = cv.v_codes + (tile_token(tile) / kTileTokens * 64 + lane) * WPL;
                keep_weights(s);
#pragma unroll 1
                for (int v = 0; v < 16; ++v) {
                    const int t = 8 * (v >> 2) + 4 * hh + (v & 3);        // slab v >> 3, pair (v >> 1) & 3, half-word v & 1
                    const float p = weights[64 * v + lane];
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const uint32_t w = BITS == 2 ? words[b] >> (8 * (v >> 3)) : words[(2 * b + (v >> 3)) % WPL];
                        const float code = (float)((w >> (BITS * ((v >> 1) & 3) + 16 * (v & 1))) & MASK);
                        const float *const m = meta + 32 * b / GROUP * 32 + t;
                        o[b] = mfma_f32((code + m[G * 32]) * m[0], p, o[b]);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (!more) break;
        }
        if constexpr (kTau) {
            tau += other_half(tau);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[b][v] += tau;
            tau = 0.0f;
        }
    }
    // The output of a wave's cached tiles (in the rotated basis) or current tiles, its maximum and sums, to slot `slot`.
    float *const red = lds + L::kRed;      // [slot][m, l_s, l_r, largest score][row]
    auto leave = [&](int slot) {
        l_s += other_half(l_s);
        l_r += other_half(l_r);
        if (hh == 0) {
            red[(slot * 4) * 32 + n] = above == -INFINITY ? -INFINITY : base;
            red[(slot * 4 + 1) * 32 + n] = l_s;
            red[(slot * 4 + 2) * 32 + n] = l_r;
            red[(slot * 4 + 3) * 32 + n] = base + above;
        }
        float *const dst = lds + (slot < kFWaves ? slot * L::kSlot : L::kSlot8) + 4 * lane;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                *reinterpret_cast<float4 *>(dst + (4 * b + g4) * L::kQuad) = float4{o[b][4 * g4], o[b][4 * g4 + 1], o[b][4 * g4 + 2], o[b][4 * g4 + 3]};
    };

    // ---- current tiles
    if (x < x_end) {
        if (!kBf16) slack = 0.0f;     // (fp32 values are asked for behind the weights)
        if (run_start(wave) < tc) {
            leave(kFWaves);
            above = -INFINITY;
            base = l_s = l_r = 0.0f;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[b][v] = 0.0f;
        }
        const T *const q_ptr = q_all + row * a.q_stride_token + (int64_t)qhead * a.q_stride_head + 8 * hh;
        const T *k_base = static_cast<const T *>(a.k_cur) + (int64_t)head * a.stride_head + 8 * hh;
        const T *v_base = static_cast<const T *>(a.v_cur) + (int64_t)head * a.stride_head;
        constexpr int kVPieces = DIM / 16;       // 16-byte pieces of a value tile per lane
        u32x4 q_raw[kBf16 ? NI : 1];             // BF16: queries as they are, lane (row, hh): channels 16 i + 8 hh + e
        if constexpr (kBf16) {
#pragma unroll
            for (int i = 0; i < NI; ++i) q_raw[i] = *reinterpret_cast<const u32x4 *>(q_ptr + 16 * i);
        }
        const int64_t last = a.n_cur - 1;
        // BF16: a tile's keys and values as they lie in memory, requested one tile ahead (keys of head_dim 128 are not:
        // no registers left); past the last key the last key's, which gets weight 0
        u32x4 k_op[kBf16 ? NI : 1], v_rows[kBf16 ? kVPieces : 1];
        auto request_keys = [&](int tile) {
            const int64_t key0 = (int64_t)(tile - tc) * kTileTokens, key = key0 + n < last ? key0 + n : last;
            const T *const kp = k_base + key * a.stride_token;
#pragma unroll
            for (int i = 0; i < NI; ++i) k_op[i % (kBf16 ? NI : 1)] = *reinterpret_cast<const u32x4 *>(kp + 16 * i);
        };
        auto request_values = [&](int tile) {
            const int64_t key0 = (int64_t)(tile - tc) * kTileTokens;
#pragma unroll
            for (int i = 0; i < kVPieces; ++i) {
                const int64_t tok = key0 + (lane + 64 * i) / (DIM / 8);
                v_rows[i % (kBf16 ? kVPieces : 1)] = *reinterpret_cast<const u32x4 *>(v_base + (tok < last ? tok : last) * a.stride_token + 8 * (lane % (DIM / 8)));
            }
        };
        if constexpr (kBf16) {
            if (DIM == 64) request_keys(x);
            request_values(x);
        }
        for (; x < x_end; ++x) {
            const int64_t key0 = (int64_t)(x - tc) * kTileTokens, key = key0 + n < last ? key0 + n : last;
            const int tok_max = __builtin_amdgcn_readfirstlane((int)(last - key0 < kTileTokens - 1 ? last - key0 : kTileTokens - 1));
            const T *const v_tile = v_base + key0 * a.stride_token;
            const T *const kp = k_base + key * a.stride_token;
            auto fp32_scores = [&](f32x16 &s) {
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = 0.0f;
#pragma unroll 1
                for (int i = 0; i < NI; ++i) {
                    float ky[8], qy[8];
                    load8(kp + 16 * i, ky);
                    load8(q_ptr + 16 * i, qy);
#pragma unroll
                    for (int e = 0; e < 8; ++e) s = mfma_f32(ky[e], qy[e] * c_log, s);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] -= base;
            };
            // fp32: values of the eight tokens of slab sl that this lane half holds, channel 32 b + n (weight 0 past the last key)
            constexpr bool kAhead = DIM == 64;      // (head_dim 128 has no registers for it)
            float vals[kAhead ? 2 : 1][NB][8];
            auto request = [&](int sl) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int tok = 16 * sl + 8 * (e >> 2) + 4 * hh + (e & 3);
                    const T *vp = v_tile + (tok <= tok_max ? tok : tok_max) * a.stride_token + n;
#pragma unroll
                    for (int b = 0; b < NB; ++b) vals[kAhead ? sl : 0][b][e] = Io<T>::load(vp + 32 * b);
                }
            };
            f32x16 s;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = 0.0f;
            if constexpr (kBf16) {
                if (DIM == 128) request_keys(x);
#pragma unroll
                for (int i = 0; i < NI; ++i) s = mfma_bf16(k_op[i], q_raw[i], s);
                if (DIM == 64 && x + 1 < x_end) request_keys(x + 1);
                float size = 0.0f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    size += fabsf(s[v]);
                    s[v] = fmaf(s[v], c_log, -base);
                }
                if (__builtin_expect(__any(!(size < INFINITY)), 0)) fp32_scores(s);   // (queries that carry the scale may stay within range)
            } else {
                if (kAhead) request(0);
                float size = 0.0f;
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    float y[8];
                    load8(kp + 16 * i, y);
                    u32x4 op[3], query[3];
#pragma unroll
                    for (int p = 0; p < 3; ++p) query[p] = *reinterpret_cast<const u32x4 *>(pieces + L::kPlain + 4 * ((p * NI + i) * 64 + lane));
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        size += fabsf(y[2 * p]) + fabsf(y[2 * p + 1]);
                        const Pieces t = split3(y[2 * p], y[2 * p + 1]);
                        set(op[0], p, t.hi);
                        set(op[1], p, t.mid);
                        set(op[2], p, t.lo);
                    }
                    s = mfma_pieces(op, query, s);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] -= base;
                if (__builtin_expect(unfit || !__all(in_range(size, kTopFactor)), 0)) fp32_scores(s);
            }
            if (a.causal || key0 + kTileTokens > a.n_cur) {
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = key0 + 8 * (v >> 2) + 4 * hh + (v & 3) < visible ? s[v] : -INFINITY;
            }
            // The rows of a tile share its values, and the weight 0 of a key that a row does not see must not meet an infinity
            // or a NaN: what is not finite goes into the product as 0 and is added below to the rows that see it.
            bool finite = true, large = false;
            if constexpr (kBf16) {
                auto beyond = [&](int limit) {
                    typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;
                    u16x2 top = {0, 0};
#pragma unroll
                    for (int i = 0; i < kVPieces; ++i) {
                        const uint32_t ws[4] = {v_rows[i].x, v_rows[i].y, v_rows[i].z, v_rows[i].w};
#pragma unroll
                        for (int j = 0; j < 4; ++j) top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, ws[j] & 0x7fff7fffu));
                    }
                    return __any(top.x >= limit || top.y >= limit);
                };
                constexpr int kLarge = (127 + 100) << 7;       // 2^100
                if (__builtin_expect(beyond(kLarge), 0)) {
                    finite = !beyond(0x7f80);
                    auto only_finite = [](uint32_t w) {
                        return (w & ((w & 0x7f80u) == 0x7f80u ? 0xffff0000u : ~0u)) & ((w & 0x7f800000u) == 0x7f800000u ? 0xffffu : ~0u);
                    };
#pragma unroll
                    for (int i = 0; i < kVPieces; ++i)
                        v_rows[i] = u32x4{only_finite(v_rows[i].x), only_finite(v_rows[i].y), only_finite(v_rows[i].z), only_finite(v_rows[i].w)};
                    large = beyond(kLarge);
                }
            }
            weigh(s, l_r, large);
            if constexpr (kBf16) {
                // Rows of the tile through LDS: the transposing read hands a lane four tokens of its channel (of 16 lanes, lane
                // 4 j + c supplies the address of token j, channels 4 c .. 4 c + 3, and lane i receives channel i).
                uint16_t *const stage = reinterpret_cast<uint16_t *>(lds + L::kOwn + wave * L::kOwnWave);
#pragma unroll
                for (int i = 0; i < kVPieces; ++i)
                    *reinterpret_cast<u32x4 *>(stage + (lane + 64 * i) / (DIM / 8) * L::kStageRow + 8 * (lane % (DIM / 8))) = v_rows[i];
                if (x + 1 < x_end) request_values(x + 1);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const uint16_t *const src = stage + (4 * hh + ((lane >> 2) & 3)) * L::kStageRow + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    u32x4 pp[3];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const Pieces t = split3(s[8 * sl + 2 * i], s[8 * sl + 2 * i + 1]);
                        set(pp[0], i, t.hi);
                        set(pp[1], i, t.mid);
                        set(pp[2], i, t.lo);
                    }
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const u32x2 t0 = read_transposed(src + 16 * sl * L::kStageRow + 32 * b), t1 = read_transposed(src + (16 * sl + 8) * L::kStageRow + 32 * b);
                        const u32x4 op = {t0.x, t0.y, t1.x, t1.y};
#pragma unroll
                        for (int p = 2; p >= 0; --p) o[b] = mfma_bf16(op, pp[p], o[b]);
                    }
                }
                __builtin_amdgcn_wave_barrier();
            } else {
                if (kAhead) request(1);
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    if (!kAhead) request(sl);
                    float (&x8)[NB][8] = vals[kAhead ? sl : 0];
                    bool fits = true;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        float size = 0.0f;
#pragma unroll
                        for (int e = 0; e < 8; ++e) size += fabsf(x8[b][e]);
                        fits = fits && in_range(size, kTop);
                    }
                    if (__builtin_expect(!__all(fits), 0)) {
                        fits = true;
                        bool all = true;
#pragma unroll
                        for (int b = 0; b < NB; ++b) {
                            float size = 0.0f;
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                if (__builtin_amdgcn_classf(x8[b][e], kNotFinite)) {
                                    all = false;
                                    x8[b][e] = 0.0f;
                                }
                                size += fabsf(x8[b][e]);
                            }
                            fits = fits && in_range(size, kTop);
                        }
                        finite = finite && __all(all);
                    }
                    if (__builtin_expect(__all(fits), 1)) {
                        u32x4 pp[3];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const Pieces t = split3(s[8 * sl + 2 * i], s[8 * sl + 2 * i + 1]);
                            set(pp[0], i, t.hi);
                            set(pp[1], i, t.mid);
                            set(pp[2], i, t.lo);
                        }
#pragma unroll
                        for (int b = 0; b < NB; ++b) {
                            u32x4 op[3];
#pragma unroll
                            for (int p = 0; p < 4; ++p) {
                                const Pieces t = split3(x8[b][2 * p], x8[b][2 * p + 1]);
                                set(op[0], p, t.hi);
                                set(op[1], p, t.mid);
                                set(op[2], p, t.lo);
                            }
                            o[b] = mfma_pieces(op, pp, o[b]);
                        }
                    } else {
                        keep_weights(s);
#pragma unroll 1
                        for (int v = 8 * sl; v < 8 * sl + 8; ++v) {
                            const int tok = 8 * (v >> 2) + 4 * hh + (v & 3);
                            const T *vp = v_tile + (tok <= tok_max ? tok : tok_max) * a.stride_token + n;
                            const float p = weights[64 * v + lane];
#pragma unroll
                            for (int b = 0; b < NB; ++b) {
                                const float w = Io<T>::load(vp + 32 * b);
                                o[b] = mfma_f32(__builtin_amdgcn_classf(w, kNotFinite) ? 0.0f : w, p, o[b]);
                            }
                        }
                    }
                }
            }
            if (__builtin_expect(!finite, 0)) {
#pragma unroll 1
                for (int tok = 0; tok <= tok_max; ++tok) {
                    const bool sees = key0 + tok < visible;
                    const T *vp = v_tile + tok * a.stride_token + 4 * hh;   // the lane's channels: 32 b + 8 g4 + 4 hh + r
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const float vv = Io<T>::load(vp + 32 * b + 8 * (v >> 2) + (v & 3));
                            o[b][v] += sees && __builtin_amdgcn_classf(vv, kNotFinite) ? vv : 0.0f;
                        }
                }
            }
        }
    }

    // ---- the workgroup's waves: their outputs, maxima and sums meet in LDS and each thread adds up its eight channels; what
    // comes from cached tiles is rotated back once, as a sum.
    __syncthreads();                       // the working areas are done with
    if (run_start(wave) < x_end) leave(wave);
    __syncthreads();
    if (!has_octet) return;
    // waves before `cached` had cached tiles only; `mixed`: wave `cached` had both kinds
    const int busy = each > 0 ? kFWaves : left;
    int cached = 0;
    while (cached < busy && run_start(cached + 1) <= tc) ++cached;
    const bool mixed = cached < busy && run_start(cached) < tc;
    const float *const my_red = red + r8;
    float top = mixed ? my_red[kFWaves * 128 + 96] : -INFINITY;
    for (int w = 0; w < busy; ++w) top = fmaxf(top, my_red[w * 128 + 96]);
    l_s = l_r = 0.0f;
    float y[8] = {}, z[8] = {};
    auto add = [&](int slot, float (&sum)[8]) {
        // (a slot without a key that the row sees has m = -inf and l = 0; if all do, or every score is -inf, all weights are 0)
        const float m = my_red[slot * 128], f = m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m - top);
        l_s = fmaf(f, my_red[slot * 128 + 32], l_s);
        l_r = fmaf(f, my_red[slot * 128 + 64], l_r);
        const float *const src = lds + (slot < kFWaves ? slot * L::kSlot : L::kSlot8) + g8 * L::kQuad + 4 * r8;
        const float4 c0 = *reinterpret_cast<const float4 *>(src), c1 = *reinterpret_cast<const float4 *>(src + 128);
        if (m == -INFINITY) return;
        sum[0] = fmaf(f, c0.x, sum[0]); sum[1] = fmaf(f, c0.y, sum[1]); sum[2] = fmaf(f, c0.z, sum[2]); sum[3] = fmaf(f, c0.w, sum[3]);
        sum[4] = fmaf(f, c1.x, sum[4]); sum[5] = fmaf(f, c1.y, sum[5]); sum[6] = fmaf(f, c1.z, sum[6]); sum[7] = fmaf(f, c1.w, sum[7]);
    };
    for (int w = 0; w < cached; ++w) add(w, y);
    if (mixed) add(kFWaves, y);
    for (int w = cached; w < busy; ++w) add(w, z);
    if (cached > 0 || mixed) {
        hadamard(y);
        const uint32_t sg = has_signs(cv) ? sign_bits_from(cv, 8 * g8) : 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] += flip_sign(y[e] * kNorm, (sg >> e) & 1u);
    }
    if (block_row0 + r8 >= rows) return;
    if (piece < 0) {
        const float inv = 1.0f / (l_s + l_r);
        T *dst = static_cast<T *>(a.out) + (int64_t)qhead8 * a.q_stride_head + row8 * a.q_stride_token + 8 * g8;
        store4(dst, z[0] * inv, z[1] * inv, z[2] * inv, z[3] * inv);
        store4(dst + 4, z[4] * inv, z[5] * inv, z[6] * inv, z[7] * inv);
        if (a.mass_cached && g8 == 0) a.mass_cached[(int64_t)qhead8 * a.m + row8] = l_s * inv;
    } else {
        float4 *const dst = reinterpret_cast<float4 *>(sp.part_o) + (int64_t)piece * (DIM * 8) + g8 * 64 + r8;
        dst[0] = float4{z[0], z[1], z[2], z[3]};
        dst[32] = float4{z[4], z[5], z[6], z[7]};
        if (g8 == 0) sp.part_ml[(int64_t)piece * 32 + r8] = float4{top, l_s, l_r, 0.0f};
    }
}

template <int DIM, int BITS, typename T, bool FP8, int GROUP>
hipError_t launch_f32(const AttentionArgs &a, const SplitArgs &sp, hipStream_t stream)
{
    constexpr size_t kBytes = F32Lds<DIM, DIM / GROUP, sizeof(T) == 2>::kWords * sizeof(float);
    static std::atomic<uint64_t> configured{0};
    const auto kernel = attention_f32_kernel<DIM, BITS, T, FP8, GROUP>;
    const hipError_t e = configure_dynamic_lds(reinterpret_cast<const void *>(kernel), kBytes, configured);
    if (e != hipSuccess) return e;
    return launch_kernel(kernel, dim3((unsigned)(sp.whole + sp.pieces)), dim3(64 * kFWaves), kBytes, stream, a, sp);
}
template <int DIM, int BITS, typename T> hipError_t launch_format(const AttentionArgs &a, const SplitArgs &sp, hipStream_t stream)
{
    if (a.cv.meta_format == KVQ_META_FP32) return launch_f32<DIM, BITS, T, false, DIM>(a, sp, stream);
    if (a.cv.group_size == 32) return launch_f32<DIM, BITS, T, true, 32>(a, sp, stream);
    if (a.cv.group_size == 64) return launch_f32<DIM, BITS, T, true, 64>(a, sp, stream);
    if constexpr (DIM == 128) return launch_f32<DIM, BITS, T, true, 128>(a, sp, stream);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_attention_f32(const AttentionArgs &a, const SplitArgs &sp, hipStream_t stream)
{
    if (a.cv.key_axis != KVQ_KEYS_PER_TOKEN || a.correction > 1) return hipErrorInvalidValue;
    const bool bf16 = a.cv.io_dtype == KVQ_BF16;
    if (a.cv.head_dim == 64 && a.cv.bits == 2) return bf16 ? launch_format<64, 2, uint16_t>(a, sp, stream) : launch_format<64, 2, float>(a, sp, stream);
    if (a.cv.head_dim == 64 && a.cv.bits == 4) return bf16 ? launch_format<64, 4, uint16_t>(a, sp, stream) : launch_format<64, 4, float>(a, sp, stream);
    if (a.cv.head_dim == 128 && a.cv.bits == 2) return bf16 ? launch_format<128, 2, uint16_t>(a, sp, stream) : launch_format<128, 2, float>(a, sp, stream);
    if (a.cv.head_dim == 128 && a.cv.bits == 4) return bf16 ? launch_format<128, 4, uint16_t>(a, sp, stream) : launch_format<128, 4, float>(a, sp, stream);
    return hipErrorInvalidValue;
}

}  // namespace kvq
