// fp32 matrix-core chunk attention: every cache with one (scale, zero-point) per token or group of channels, head_dim 64
// or 128, BF16 or FP32 tensors: the caches that the 16-bit kernels do not serve, and calls with a few query rows, which
// would leave most of their 256-row blocks empty.  All inputs of the matrix instructions are fp32 and so is everything computed from them
// (v_mfma_f32_32x32x2_f32), so the results have the precision of the vector kernel, whose arithmetic this is: keys and
// values are reconstructed as (code - zero) * scale, scored against the rotated query, corrected by
// b = sigma^2 / 24 * sum_j step_j^2 nu_j.
//
// Work split.  A unit is 32 query rows of one query head (or of the query heads that share a key/value head, one after
// the other: four heads with a row each are one unit and read the cache once); a workgroup of 8 wavefronts (two per SIMD: one unpacks while
// the other multiplies) takes a unit, or a piece of its key range, and deals its 32-key tiles to the wavefronts in turn.
// Each wavefront keeps its own maximum, sums and output tile; they are put together through LDS at the end.  Few rows
// (one token behind a long prefix) thereby still keep a compute unit busy, and no wavefront waits for another until then.
//
// Operands.  Everything is transposed, S^T = K Q^T and O^T = V^T P^T: a lane owns query row lane mod 32 of both result
// tiles.  The packed layout hands each lane exactly the codes it feeds to the A operand (key lane (t, hh): the channels with
// bit 3 = hh of token t; value lane (c, hh): the tokens with bit 2 = hh of channels c, c + 32, ..), so codes go from memory
// to registers to MFMA, without LDS.  Order of the contraction over channels: MFMA 8 i + e multiplies channels 16 i + e
// (lanes 0..31) and 16 i + 8 + e (lanes 32..63); over tokens: MFMA v multiplies tokens 8 (v >> 2) + (v & 3) and that + 4,
// the two keys whose scores the lane halves hold in result register v, so probabilities are B operands as they stand.
// The correction is one or two more MFMAs of the score: squared steps against -sigma^2 / 24 nu_j.
//
// Bound by the fp32 matrix rate (157 TFLOP/s nominal; 64 clocks per MFMA and SIMD), next to which unpacking takes 4
// vector instructions per code.  Why this shape: the vector kernel before it ran one row per workgroup with every key
// decoded per row, 1.6 TFLOP/s.  12 heads x 500 rows x (1500 + 500) keys, head_dim 64: 1964 -> 51 us (60 TFLOP/s; 192
// workgroups, 38 % of the fp32 matrix rate).  1 head x 64 rows x (256 + 64) keys in fp32, append included: 112 -> 22 us.
#include "kvq_internal.h"

namespace kvq {
namespace {
#include "kvq_mfma_common.h"

constexpr int kFWaves = 8, kFRows = 32;
constexpr int kNotFinite = 0x207;   // class mask: either NaN, either infinity
constexpr float kMaxFinite = 3.4028234664e38f;

// value of the other lane half
__device__ inline float other_half(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}
__device__ inline f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

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
__device__ inline void store4(float *p, float a, float b, float c, float d) { *reinterpret_cast<float4 *>(p) = float4{a, b, c, d}; }
__device__ inline void store4(uint16_t *p, float a, float b, float c, float d)
{
    *reinterpret_cast<uint2 *>(p) = uint2{(uint32_t)float_to_bf16(a) | ((uint32_t)float_to_bf16(b) << 16),
                                          (uint32_t)float_to_bf16(c) | ((uint32_t)float_to_bf16(d) << 16)};
}

// Words of LDS: value metadata of each wave's tile [wave][scale | zero][group][token], later the outputs of half the waves.
template <int DIM> constexpr int f32_lds_words()
{
    const int meta = kFWaves * 2 * 4 * 32, merge = (kFWaves / 2) * DIM * 32;
    return (meta > merge ? meta : merge) + kFWaves * 32 * 3;
}

// GROUP: channels per (scale, zero-point); DIM and fp32 pairs for KVQ_META_FP32, FP8: E4M3 / BF16 encodings.
template <int DIM, int BITS, typename T, bool FP8, int GROUP>
__global__ __launch_bounds__(64 * kFWaves, 2) void attention_f32_kernel(AttentionArgs a, SplitArgs sp)
{
    constexpr int WPL = DIM * BITS / 64;          // words of a lane's codes per tile
    constexpr int NI = DIM / 16, NB = DIM / 32;   // channel slabs of the score, channel blocks of the output
    constexpr int G = DIM / GROUP;
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    constexpr float kNorm = DIM == 64 ? 0.125f : 0.088388347648318f;
    __shared__ __align__(16) float lds[f32_lds_words<DIM>()];
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
    const int64_t packed_row = block_row0 + n < rows ? block_row0 + n : rows - 1;
    const bool row_valid = block_row0 + n < rows;
    int64_t row = packed_row;
    int qhead = qhead0;
    if (sp.pack > 1) {
        qhead += (int)((uint32_t)packed_row / (uint32_t)a.m);
        row = (uint32_t)packed_row % (uint32_t)a.m;
    }
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
    const int x0 = piece < 0 ? 0 : (int)((int64_t)all * split / sp.splits);
    const int x1 = piece < 0 ? all : (int)((int64_t)all * (split + 1) / sp.splits);
    const int first_off = (int)(a.cache_start - t_first * kTileTokens);

    // ---- query: lane (row, hh) holds channels 16 i + 8 hh + e in q[8 i + e]
    const T *q_ptr = static_cast<const T *>(a.q) + row * a.q_stride_token + (int64_t)qhead * a.q_stride_head + 8 * hh;
    const float c_log = a.softmax_scale * kLog2e;
    float q[8 * NI], corr[(G + 1) / 2];
    auto load_query = [&]() {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            float x[8];
            load8(q_ptr + 16 * i, x);
#pragma unroll
            for (int e = 0; e < 8; ++e) q[8 * i + e] = x[e];
        }
    };
    auto rotate_query = [&]() {
        load_query();
        if (has_signs(cv))
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const uint32_t sg = sign_bits_from(cv, 16 * i) >> (8 * hh);
#pragma unroll
                for (int e = 0; e < 8; ++e) q[8 * i + e] = flip_sign(q[8 * i + e], sg >> e);
            }
#pragma unroll
        for (int h = 1; h < 8 * NI; h <<= 1)
#pragma unroll
            for (int i = 0; i < 8 * NI; ++i)
                if ((i & h) == 0) {
                    const float p = q[i], r = q[i + h];
                    q[i] = p + r;
                    q[i + h] = p - r;
                }
#pragma unroll
        for (int i = 0; i < 8 * NI; ++i) {
            const float o = other_half(q[i]);
            q[i] = (hh ? o - q[i] : q[i] + o) * kNorm;
        }
        float nu[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            float s = 0.0f;
#pragma unroll
            for (int i = 0; i < 8 * NI / G; ++i) s = fmaf(q[j * (8 * NI / G) + i], q[j * (8 * NI / G) + i], s);
            nu[j] = s + other_half(s);
        }
#pragma unroll
        for (int j = 0; j < (G + 1) / 2; ++j) {
            const float second = 2 * j + 1 < G ? nu[(2 * j + 1) % G] : 0.0f;
            corr[j] = a.correction == 1 ? -(hh ? second : nu[2 * j]) * (a.softmax_scale * c_log * (1.0f / 24.0f)) : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < 8 * NI; ++i) q[i] *= c_log;
    };

    f32x16 o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[b][v] = 0.0f;
    float m_ref = -INFINITY, l_s = 0.0f, l_r = 0.0f;

    // s: scores in log2 units (-inf: key not seen) -> weights; moves the maximum
    auto weigh = [&](f32x16 &s, float &l) {
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        mx = fmaxf(mx, other_half(mx));
        if (__any(mx > m_ref)) {
            const float top = fmaxf(m_ref, mx);
            const float alpha = m_ref == top ? 1.0f : __builtin_amdgcn_exp2f(m_ref - top);
            l_s *= alpha;
            l_r *= alpha;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[b][v] *= alpha;
            m_ref = top;
        }
        const float base = m_ref == -INFINITY ? 0.0f : m_ref;
        float sum = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(s[v] - base);
            sum += s[v];
        }
        l += sum;
    };

    // ---- cached tiles
    int x = x0 + wave;
    if (x < x1 && x < tc) {
        rotate_query();
        const int64_t cap = cv.cap_tiles, head_tile0 = (int64_t)head * cap;
        float *const meta = lds + wave * (2 * G * 32);      // this wave's value metadata: [scale | zero][group][token]
        const float off = code_offset(BITS);
        uint32_t kw[WPL], vw[WPL];
        float ks[G], kz[G], vs[G], vz[G];
        bool seen;
        auto fetch = [&](int tile) {
            int64_t phys = a.phys_tile_first + tile;        // a window has at most cap + 1 tiles
            phys -= phys >= cap ? cap : 0;
            phys -= phys >= cap ? cap : 0;
            const int64_t word = ((head_tile0 + phys) * 64 + lane) * WPL;
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
            const int64_t tok = (head_tile0 + phys) * kTileTokens + n;
#pragma unroll
            for (int j = 0; j < G; ++j) {
                if constexpr (FP8) {
                    ks[j] = e4m3_low_byte(cv.k_scale8[tok * G + j]);
                    vs[j] = e4m3_low_byte(cv.v_scale8[tok * G + j]);
                    kz[j] = bf16_to_float(cv.k_zero16[tok * G + j]);
                    vz[j] = bf16_to_float(cv.v_zero16[tok * G + j]);
                } else {
                    ks[j] = cv.k_scale[tok];
                    vs[j] = cv.v_scale[tok];
                    kz[j] = -cv.k_negzero[tok] - off;
                    vz[j] = cv.v_zero_off[tok] - off;
                }
            }
        };
        fetch(x);
        for (;;) {
            // this tile's operands; the next tile's words are requested as soon as they are free
            const int tile = x;
            const bool edge = tile == 0 || tile == tc - 1;
            if (!seen) {
#pragma unroll
                for (int j = 0; j < G; ++j) ks[j] = kz[j] = vs[j] = vz[j] = 0.0f;
            }
#pragma unroll
            for (int j = 0; j < G; ++j) meta[(hh * G + j) * 32 + n] = hh ? vz[j] : vs[j];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            f32x16 s;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = 0.0f;
            // The square of an fp32 step overflows beyond 2^64, where the correction can be ordinary (tiny queries) or off:
            // tiles with such a step take it factor by factor, as the vector kernel does.  (FP8 steps end at 448.)
            if (!FP8 && __builtin_expect(__any(ks[0] >= 0x1p64f), 0)) {
                const float upper = other_half(corr[0]), c = hh ? upper : corr[0];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float st = __shfl(ks[0], 8 * (v >> 2) + 4 * hh + (v & 3));
                    s[v] = c * st * st;
                }
            } else {
#pragma unroll
                for (int j = 0; j < (G + 1) / 2; ++j) {
                    const float second = 2 * j + 1 < G ? ks[(2 * j + 1) % G] : 0.0f;
                    const float st = hh ? second : ks[2 * j];
                    s = mfma_f32(st * st, corr[j], s);
                }
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const uint32_t w = BITS == 2 ? kw[i >> 1] >> (8 * (i & 1)) : kw[i];
                const float scale = ks[16 * i / GROUP], zero = kz[16 * i / GROUP];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float code = (float)((w >> (BITS * (e >> 1) + 16 * (e & 1))) & MASK);
                    s = mfma_f32((code - zero) * scale, q[8 * i + e], s);
                }
            }
            uint32_t vcur[WPL];
#pragma unroll
            for (int i = 0; i < WPL; ++i) vcur[i] = vw[i];
            x += kFWaves;
            const bool more = x < x1 && x < tc;
            if (more) fetch(x);
            if (edge) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int rel = tile * kTileTokens + 8 * (v >> 2) + 4 * hh + (v & 3) - first_off;
                    s[v] = rel >= 0 && rel < a.cache_len ? s[v] : -INFINITY;
                }
            }
            weigh(s, l_s);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const float *msrc = meta + (32 * b / GROUP) * 32 + 4 * hh;
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const float4 sc = *reinterpret_cast<const float4 *>(msrc + 8 * g4);
                    const float4 zc = *reinterpret_cast<const float4 *>(msrc + G * 32 + 8 * g4);
                    const float scs[4] = {sc.x, sc.y, sc.z, sc.w}, zcs[4] = {zc.x, zc.y, zc.z, zc.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // token 8 g4 + 4 hh + r: slab g4 >> 1, register 2 (g4 & 1) + (r >> 1), half-word r & 1
                        const int reg = 2 * (g4 & 1) + (r >> 1), sl = g4 >> 1;
                        const uint32_t w = BITS == 2 ? vcur[b] >> (8 * sl) : vcur[(2 * b + sl) % WPL];
                        const float code = (float)((w >> (BITS * reg + 16 * (r & 1))) & MASK);
                        o[b] = mfma_f32((code - zcs[r]) * scs[r], s[4 * g4 + r], o[b]);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (!more) break;
        }
        // back from the rotated basis: channel of register (b, v) is 32 b + 8 (v >> 2) + 4 hh + (v & 3)
#pragma unroll
        for (int h = 1; h < 16; h <<= 1)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if ((v & h) == 0) {
                        const float p = o[b][v], r = o[b][v + h];
                        o[b][v] = p + r;
                        o[b][v + h] = p - r;
                    }
#pragma unroll
        for (int h = 1; h < NB; h <<= 1)
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if ((b & h) == 0) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float p = o[b][v], r = o[b + h][v];
                        o[b][v] = p + r;
                        o[b + h][v] = p - r;
                    }
                }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint32_t sg = has_signs(cv) ? cv.sign_mask[b] >> (4 * hh) : 0u;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float r = other_half(o[b][v]);
                o[b][v] = flip_sign((hh ? r - o[b][v] : o[b][v] + r) * kNorm, sg >> (8 * (v >> 2) + (v & 3)));
            }
        }
    }

    // ---- current tiles
    if (x < x1) {
        load_query();
#pragma unroll
        for (int i = 0; i < 8 * NI; ++i) q[i] *= c_log;
        const T *k_base = static_cast<const T *>(a.k_cur) + (int64_t)head * a.stride_head + 8 * hh;
        const T *v_base = static_cast<const T *>(a.v_cur) + (int64_t)head * a.stride_head + n;
        for (; x < x1; x += kFWaves) {
            const int64_t key0 = (int64_t)(x - tc) * kTileTokens;
            const int64_t last = a.n_cur - 1, key = key0 + n < last ? key0 + n : last;
            f32x16 s;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = 0.0f;
            const int tok_max = (int)(last - key0 < kTileTokens - 1 ? last - key0 : kTileTokens - 1);
            const T *const v_tile = v_base + key0 * a.stride_token;
            const T *kp = k_base + key * a.stride_token;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                float kx[8];
                load8(kp + 16 * i, kx);
#pragma unroll
                for (int e = 0; e < 8; ++e) s = mfma_f32(kx[e], q[8 * i + e], s);
            }
            if (a.causal || key0 + kTileTokens > a.n_cur) {
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = key0 + 8 * (v >> 2) + 4 * hh + (v & 3) < visible ? s[v] : -INFINITY;
            }
            weigh(s, l_r);
            // The rows of a tile share its values, and the weight 0 of a key that a row does not see must not meet an infinity
            // or a NaN: values go into the product limited to finite ones (a NaN comes out of the limits as one of them),
            // and what was not finite is added below to the rows that see it.
            // (The values of two tokens are requested ahead of the two in work: left to itself the compiler waits for every
            // load of this form, 44 us in place of 39 us for 8 x 4 heads x 1 row x (8192 + 64) keys.)
            float nan_if_found = 0.0f;
            T vals[2][2][NB];
            auto request = [&](int v, T (&into)[2][NB]) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int tok = 8 * (v >> 2) + 4 * hh + (v & 3) + u;
                    const T *vp = v_tile + (tok <= tok_max ? tok : tok_max) * a.stride_token;   // (weight 0 past the last key)
#pragma unroll
                    for (int b = 0; b < NB; ++b) into[u][b] = vp[32 * b];
                }
            };
            request(0, vals[0]);
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                if (v < 14) request(v + 2, vals[((v >> 1) + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const float vv = Io<T>::load(&vals[(v >> 1) & 1][u][b]);
                        nan_if_found = fmaf(vv, 0.0f, nan_if_found);
                        o[b] = mfma_f32(__builtin_amdgcn_fmed3f(vv, -kMaxFinite, kMaxFinite), s[v + u], o[b]);
                    }
            }
            if (__builtin_expect(__any(nan_if_found != 0.0f), 0)) {
#pragma unroll 1
                for (int tok = 0; tok <= tok_max; ++tok) {
                    const bool sees = key0 + tok < visible;
                    const T *vp = v_tile + tok * a.stride_token - n + 4 * hh;   // the lane's channels: 32 b + 8 g4 + 4 hh + r
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

    // ---- the workgroup's waves: maximum, then weighted sums, half of the waves handing theirs to the other half
    __syncthreads();                       // the metadata areas are done with
    constexpr int kMerge = (kFWaves / 2) * DIM * 32 > kFWaves * 256 ? (kFWaves / 2) * DIM * 32 : kFWaves * 256;
    float *const red = lds + kMerge;       // [wave][m, l_s, l_r][row]
    l_s += other_half(l_s);
    l_r += other_half(l_r);
    if (hh == 0) {
        red[(wave * 3) * 32 + n] = m_ref;
        red[(wave * 3 + 1) * 32 + n] = l_s;
        red[(wave * 3 + 2) * 32 + n] = l_r;
    }
    __syncthreads();
    float top = -INFINITY;
#pragma unroll
    for (int w = 0; w < kFWaves; ++w) top = fmaxf(top, red[(w * 3) * 32 + n]);
    // (a wave that has seen no key of the row has m = -inf and l = 0; if none has, or every score is -inf, all weights are 0)
    auto weight = [&](float m) { return m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m - top); };
    l_s = l_r = 0.0f;
#pragma unroll
    for (int w = 0; w < kFWaves; ++w) {
        const float f = weight(red[(w * 3) * 32 + n]);
        l_s = fmaf(f, red[(w * 3 + 1) * 32 + n], l_s);
        l_r = fmaf(f, red[(w * 3 + 2) * 32 + n], l_r);
    }
    const float mine = weight(m_ref);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[b][v] = m_ref == -INFINITY ? 0.0f : o[b][v] * mine;
#pragma unroll
    for (int half = kFWaves / 2; half >= 1; half >>= 1) {
        if (wave >= half && wave < 2 * half) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4)
                    *reinterpret_cast<float4 *>(lds + (((wave - half) * NB + b) * 4 + g4) * 256 + 4 * lane) =
                        float4{o[b][4 * g4], o[b][4 * g4 + 1], o[b][4 * g4 + 2], o[b][4 * g4 + 3]};
        }
        __syncthreads();
        if (wave < half) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const float4 r = *reinterpret_cast<const float4 *>(lds + ((wave * NB + b) * 4 + g4) * 256 + 4 * lane);
                    o[b][4 * g4] += r.x; o[b][4 * g4 + 1] += r.y; o[b][4 * g4 + 2] += r.z; o[b][4 * g4 + 3] += r.w;
                }
        }
        __syncthreads();
    }
    if (wave != 0 || !row_valid) return;
    if (piece < 0) {
        const float inv = 1.0f / (l_s + l_r);
        T *dst = static_cast<T *>(a.out) + (int64_t)qhead * a.q_stride_head + row * a.q_stride_token + 4 * hh;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                store4(dst + 32 * b + 8 * g4, o[b][4 * g4] * inv, o[b][4 * g4 + 1] * inv, o[b][4 * g4 + 2] * inv, o[b][4 * g4 + 3] * inv);
        if (a.mass_cached && hh == 0) a.mass_cached[(int64_t)qhead * a.m + row] = l_s * inv;
    } else {
        float4 *dst = reinterpret_cast<float4 *>(sp.part_o) + (int64_t)piece * (DIM * 8) + lane;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                dst[(4 * b + g4) * 64] = float4{o[b][4 * g4], o[b][4 * g4 + 1], o[b][4 * g4 + 2], o[b][4 * g4 + 3]};
        if (hh == 0) sp.part_ml[(int64_t)piece * 32 + n] = float4{top, l_s, l_r, 0.0f};
    }
}

template <int DIM, int BITS, typename T, bool FP8, int GROUP>
hipError_t launch_f32(const AttentionArgs &a, const SplitArgs &sp, hipStream_t stream)
{
    return launch_kernel(attention_f32_kernel<DIM, BITS, T, FP8, GROUP>, dim3((unsigned)(sp.whole + sp.pieces)), dim3(64 * kFWaves), 0, stream, a, sp);
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
