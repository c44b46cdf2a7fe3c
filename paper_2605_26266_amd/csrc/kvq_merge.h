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
// CHUNK pieces' references, sums and outputs are asked for together; more pieces, CHUNK at a time under a running maximum.
// Looking for the maximum over all pieces first and for the outputs then is two waits one behind the other, each about as long as
// the transfer: calls of 16 to 23 us whose fp32 kernel is split took 1 to 3 us more (17.1 -> 14.1, 17.7 -> 15.7, 22.7 -> 21.4).
// One token behind 8192 keys, with more than 8 pieces, is the other end: 20.5 -> 20.7 us; 16 at a time were 23.1, two times 8 in
// flight 20.7.
template <int DIM, typename T, bool GATED, int CHUNK> __device__ inline bool merge_pieces(const AttentionArgs &a, const SplitArgs &sp)
{
    const int lane = threadIdx.x & 63, g = 2 * (int)(blockIdx.x & 1) + (int)(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    constexpr int NB = DIM / 32;
    const unsigned block = blockIdx.x >> 1;
    const int b = block % NB;
    const int row_block = (int)(block / NB % sp.part_blocks), unit_rel = (int)(block / NB / sp.part_blocks);
    const int64_t block0 = (int64_t)unit_rel * sp.splits * sp.part_blocks + row_block;
    // uniform addresses plus an offset per lane: no 64-bit address per load in vector registers
    const float4 *ml = sp.part_ml + block0 * 32, *po = reinterpret_cast<const float4 *>(sp.part_o) + block0 * (DIM * 8);
    const uint32_t ml_lane = (uint32_t)n, po_lane = (uint32_t)((4 * b + g) * 64 + lane);
    const int64_t ml_step = (int64_t)sp.part_blocks * 32, po_step = (int64_t)sp.part_blocks * (DIM * 8);

    const bool flagged = GATED && cache_flagged(a.status);
    float4 p[CHUNK], v[CHUNK];
    auto fetch = [&](int s0) {
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) {
            const int s = s0 + i < sp.splits ? s0 + i : sp.splits - 1;   // past the last piece: read again, left out below
            p[i] = (ml + s * ml_step)[ml_lane];
            v[i] = (po + s * po_step)[po_lane];
        }
    };
    fetch(0);
    asm volatile("" ::: "memory");   // the loads are issued here, not where they are used
    if (flagged) return false;
    const int unit = sp.whole + unit_rel;
    const int group = unit / sp.row_blocks, rblk = unit % sp.row_blocks;
    int64_t row = (int64_t)rblk * sp.rows + 32 * row_block + n;
    if (row >= a.m * sp.pack) return true;
    int qhead = group * sp.pack;
    if (sp.pack > 1) {     // (the host packs heads only where the product fits 31 bits)
        qhead += (int)((uint32_t)row / (uint32_t)a.m);
        row = (uint32_t)row % (uint32_t)a.m;
    }

    float top = -INFINITY, ls = 0.0f, lr = 0.0f;
    float4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = 0;;) {
        const float before = top;
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) top = fmaxf(top, p[i].x);
        if (s0 > 0) {
            const float alpha = before == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(before - top);
            ls *= alpha; lr *= alpha;
            acc.x *= alpha; acc.y *= alpha; acc.z *= alpha; acc.w *= alpha;
        }
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) {
            const bool none = (p[i].x == -INFINITY && p[i].y == 0.0f && p[i].z == 0.0f) || s0 + i >= sp.splits;
            const float w = none ? 0.0f : __builtin_amdgcn_exp2f(p[i].x - top);
            ls = none ? ls : fmaf(w, p[i].y, ls);
            lr = none ? lr : fmaf(w, p[i].z, lr);
            acc.x = none ? acc.x : fmaf(w, v[i].x, acc.x);
            acc.y = none ? acc.y : fmaf(w, v[i].y, acc.y);
            acc.z = none ? acc.z : fmaf(w, v[i].z, acc.z);
            acc.w = none ? acc.w : fmaf(w, v[i].w, acc.w);
        }
        s0 += CHUNK;
        if (s0 >= sp.splits) break;
        fetch(s0);
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
    return true;
}
// By workgroups below merge_workgroups.  GATED: behind a 16-bit launch, which stands back on a flagged cache: false then, and
// nothing written (the pieces are read all the same: the work space is there).
template <int DIM, typename T, bool GATED> __device__ inline bool merge_rows(const AttentionArgs &a, const SplitArgs &sp)
{
    if (sp.splits <= 4) return merge_pieces<DIM, T, GATED, 4>(a, sp);   // (no more loads than pieces where they are few)
    return merge_pieces<DIM, T, GATED, 8>(a, sp);
}
