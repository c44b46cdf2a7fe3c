// Combines the pieces of the units whose key range a matrix-core attention launch has split (SplitArgs).
//
// For every row: M = max over pieces of the reference m_i, w_i = 2^(m_i - M),
//     out = sum_i w_i O_i / sum_i w_i (l_s,i + l_r,i),   mass = sum_i w_i l_s,i / the same,
// all in fp32.  A piece without a key that the row sees carries m_i = -inf and l_i = 0 and is left out.
//
// Bound by the partial outputs, 16 KiB per piece and 32 rows, which come out of the L2 / Infinity Cache they have just
// been written to.  One wave per 32 rows, channel block and register quad: a load instruction of a wave is 1 KiB in one
// run, and a call with a few rows and many pieces (one new token behind a long prefix) still has 16 waves per 32 rows,
// so the pieces' loads are in flight together instead of one behind the other.
// Included inside namespace kvq { namespace { ... } }.
#pragma once

constexpr int kMergeThreads = 128;   // two register quads of one 32-row block and channel block
template <int DIM> inline unsigned merge_workgroups(const SplitArgs &sp)
{
    return (unsigned)(sp.pieces / sp.splits * sp.part_blocks) * (DIM / 32) * 2;   // at most 1024 units of 8 blocks
}
// (by workgroups below merge_workgroups)
template <int DIM, typename T> __device__ inline void merge_rows(const AttentionArgs &a, const SplitArgs &sp)
{
    const int lane = threadIdx.x & 63, g = 2 * (int)(blockIdx.x & 1) + (int)(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    constexpr int NB = DIM / 32;
    const unsigned block = blockIdx.x >> 1;
    const int b = block % NB;
    const int row_block = (int)(block / NB % sp.part_blocks), unit_rel = (int)(block / NB / sp.part_blocks);
    const int unit = sp.whole + unit_rel;
    const int group = unit / sp.row_blocks, rblk = unit % sp.row_blocks;
    int64_t row = (int64_t)rblk * sp.rows + 32 * row_block + n;
    if (row >= a.m * sp.pack) return;
    int qhead = group * sp.pack;
    if (sp.pack > 1) {     // (the host packs heads only where the product fits 31 bits)
        qhead += (int)((uint32_t)row / (uint32_t)a.m);
        row = (uint32_t)row % (uint32_t)a.m;
    }
    const int64_t block0 = (int64_t)unit_rel * sp.splits * sp.part_blocks + row_block;
    const float4 *ml = sp.part_ml + block0 * 32 + n;
    const float4 *po = reinterpret_cast<const float4 *>(sp.part_o) + block0 * (DIM * 8) + (4 * b + g) * 64 + lane;
    const int64_t ml_step = (int64_t)sp.part_blocks * 32, po_step = (int64_t)sp.part_blocks * (DIM * 8);

    float top = -INFINITY;
#pragma unroll 8
    for (int s = 0; s < sp.splits; ++s) top = fmaxf(top, ml[s * ml_step].x);
    float ls = 0.0f, lr = 0.0f;
    float4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
    for (int s = 0; s < sp.splits; ++s) {
        const float4 p = ml[s * ml_step];
        const float4 v = po[s * po_step];
        const bool none = p.x == -INFINITY && p.y == 0.0f && p.z == 0.0f;
        const float w = none ? 0.0f : __builtin_amdgcn_exp2f(p.x - top);
        ls = fmaf(w, p.y, ls);
        lr = fmaf(w, p.z, lr);
        acc.x = none ? acc.x : fmaf(w, v.x, acc.x);
        acc.y = none ? acc.y : fmaf(w, v.y, acc.y);
        acc.z = none ? acc.z : fmaf(w, v.z, acc.z);
        acc.w = none ? acc.w : fmaf(w, v.w, acc.w);
    }
    const float inv = 1.0f / (ls + lr);
    T *dst = static_cast<T *>(a.out) + (int64_t)qhead * a.q_stride_head + row * a.q_stride_token + 32 * b + 8 * g + 4 * hh;
    if constexpr (sizeof(T) == 2) {
        uint2 w;
        w.x = (uint32_t)float_to_bf16(acc.x * inv) | ((uint32_t)float_to_bf16(acc.y * inv) << 16);
        w.y = (uint32_t)float_to_bf16(acc.z * inv) | ((uint32_t)float_to_bf16(acc.w * inv) << 16);
        *reinterpret_cast<uint2 *>(dst) = w;
    } else {
        *reinterpret_cast<float4 *>(dst) = float4{acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv};
    }
    if (a.mass_cached && hh == 0 && b == 0 && g == 0) a.mass_cached[(int64_t)qhead * a.m + row] = ls * inv;
}
