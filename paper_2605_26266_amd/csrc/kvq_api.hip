// Host layer of the C ABI: argument validation, the cache object, dispatch to the kernels.
// No device memory is allocated here; the cache storage is carved out of the caller's buffer.
#include <deque>
#include <new>

#include "kvq_internal.h"

struct kvq_block {
    int slot;        // index into the per-block metadata arrays
    int64_t start;   // logical position of the block's first token
    int64_t count;   // tokens of the block (shrinks when the cache is truncated)
};

struct kvq_cache {
    kvq_cache_desc desc;
    kvq::CacheView view;
    int64_t cap32;  // capacity rounded up to whole tiles
    int64_t base;   // logical position of the oldest live token (the storage is a ring)
    int64_t len;    // live tokens
    std::deque<kvq_block> blocks;   // KVQ_KEYS_PER_CHANNEL: live appended blocks, oldest first
    int next_slot;
    bool status_clean;   // the status block has been cleared on the device since the cache was created or reset

    // Forget blocks that lie wholly outside [base, base + len).
    void trim_blocks()
    {
        while (!blocks.empty() && blocks.front().start + blocks.front().count <= base) blocks.pop_front();
        while (!blocks.empty() && blocks.back().start >= base + len) {   // slots stay consecutive: reuse it next
            next_slot = blocks.back().slot;
            blocks.pop_back();
        }
        if (!blocks.empty() && blocks.back().start + blocks.back().count > base + len)
            blocks.back().count = base + len - blocks.back().start;
        if (len == 0) blocks.clear();
    }
};

namespace {

kvq_status check_desc(const kvq_cache_desc *d)
{
    if (!d) return KVQ_ERR_INVALID_ARG;
    if (d->num_heads < 1 || d->capacity_tokens < 1 || d->head_dim < 1 || d->bits < 1) return KVQ_ERR_INVALID_ARG;
    if (d->io_dtype != KVQ_BF16 && d->io_dtype != KVQ_FP32) return KVQ_ERR_INVALID_ARG;
    if (d->head_dim != 64 && d->head_dim != 128) return KVQ_ERR_UNSUPPORTED;
    if (d->bits != 2 && d->bits != 4) return KVQ_ERR_UNSUPPORTED;
    if (d->meta_format != KVQ_META_FP32 && d->meta_format != KVQ_META_FP8_BF16) return KVQ_ERR_INVALID_ARG;
    if (d->group_size != d->head_dim && d->group_size != 32 && d->group_size != 64) return KVQ_ERR_UNSUPPORTED;
    if (d->group_size > d->head_dim) return KVQ_ERR_UNSUPPORTED;
    if (d->group_size != d->head_dim && d->meta_format != KVQ_META_FP8_BF16) return KVQ_ERR_UNSUPPORTED;
    if (d->rotate != 1) return KVQ_ERR_UNSUPPORTED;
    if (d->key_axis != KVQ_KEYS_PER_TOKEN && d->key_axis != KVQ_KEYS_PER_CHANNEL) return KVQ_ERR_INVALID_ARG;
    if (d->key_axis == KVQ_KEYS_PER_CHANNEL && (d->meta_format != KVQ_META_FP32 || d->group_size != d->head_dim))
        return KVQ_ERR_UNSUPPORTED;
    if (d->capacity_tokens > ((int64_t)1 << 40)) return KVQ_ERR_INVALID_ARG;
    return KVQ_OK;
}

int64_t round_up_tile(int64_t n) { return (n + kvq::kTileTokens - 1) / kvq::kTileTokens * kvq::kTileTokens; }

int64_t max_blocks_of(int64_t cap32) { return cap32 / kvq::kTileTokens + 2; }

// Bytes of the per-channel key metadata that follow the ordinary storage (0 for per-token keys).
int64_t channel_bytes(const kvq_cache_desc *d, int64_t cap32)
{
    if (d->key_axis != KVQ_KEYS_PER_CHANNEL) return 0;
    const int64_t hd = (int64_t)d->num_heads * d->head_dim;
    const int64_t n = max_blocks_of(cap32) * hd * 8 + cap32 * 4 + hd * 32;
    return (n + 255) / 256 * 256;
}

size_t elt_bytes(int io_dtype) { return io_dtype == KVQ_BF16 ? 2 : 4; }

// Tensor arguments: 16-byte aligned base, strides that keep every (token, head) vector 16-byte aligned.
bool tensor_ok(const void *p, int64_t stride_token, int64_t stride_head, int head_dim, int io_dtype)
{
    if (!p) return false;
    if (reinterpret_cast<uintptr_t>(p) % 16 != 0) return false;
    const int64_t quantum = 16 / (int64_t)elt_bytes(io_dtype);
    if (stride_token < head_dim || stride_head < head_dim) return false;
    if (stride_token % quantum != 0 || stride_head % quantum != 0) return false;
    return true;
}

// How a matrix-core call is laid over the 256 compute units (one workgroup each).  The units (row blocks) that fill whole
// rounds of the chip stay whole; the key ranges of the rest are cut into the number of pieces with the shortest estimated
// time: rounds * (tiles per piece + what a workgroup pays once: query preparation, rotation back, writing its result) + the
// merge.  The constants (microseconds) follow measurements, estimates in brackets.  8 heads x 1024 rows x (4096 + 1024) keys,
// 32 units of the per-token kernel: 175 (182) / 111 (110) / 82 (71) / 61 (54) / 84 (87) / 134 (138) us with 1 / 2 / 4 / 8 /
// 12 / 32 pieces.  32 query heads x 1 row x (8192 + 64) keys, group-wise kernel: 361 (374) / 114 (121) / 70 (78) / 87 (107) /
// 122 (165) us with 1 / 4 / 8 / 16 / 32; fp32 kernel, 8 units: 108 (108) / 39 (40) / 26 (29) / 21 (22) / 20 (23) / 21 (24) /
// 32 (42) us with 1 / 4 / 8 / 17 / 24 / 32 / 64; head_dim 64, 2 heads x 300 rows x (4000 + 300) keys, 20 units: 38 (44) / 26 (30) /
// 20 (23) / 16 (20) / 17 (18) / 30 (47) us with 1 / 2 / 4 / 8 / 12 / 32 (0.19 us a tile; fp32 tensors and groups take 0.3).  Over
// random calls (see choose()) all three estimates are high, by 5 to 20 % on average, and alike: the 16-bit kernels took 0.79 to
// 0.98 of theirs, the fp32 kernel 0.81 to 0.97.  24 heads x 4680 rows x (28080 + 4680) keys, 200 units after a full round: 2043
// (2094) / 2133 (2131) / 2044 (1982) / 2089 (2043) / 2110 (2178) us with 1 / 2 / 5 / 6 / 9.
struct KernelCost {
    int rows;          // query rows of a unit
    int threads;       // of its workgroup
    int tiles_step;    // tiles that a workgroup works on side by side
    double tile, fixed, merge;
};
constexpr KernelCost kCostPerToken{256, 256, 1, 1.0, 22.0, 6.0}, kCostGroup{256, 256, 1, 1.35, 26.0, 6.0};
constexpr KernelCost kCostF32Dim64{kvq::kF32Rows, 512, 8, 0.24, 11.0, 1.5}, kCostF32Dim128{kvq::kF32Rows, 512, 8, 0.36, 12.5, 1.5};

struct Plan {
    kvq::SplitArgs sp;
    double cost;
};
constexpr double kTooLarge = 1e300;   // more units than a grid holds

Plan plan_split(const KernelCost &k, int64_t m, int64_t heads, int64_t ratio, int64_t tiles, bool may_split)
{
    constexpr int kComputeUnits = 256, kMaxSplits = 64;
    constexpr double kMergePerSplit = 0.12, kMergePerBlock = 0.0025;
    kvq::SplitArgs sp = {};
    sp.rows = k.rows;
    sp.pack = (int32_t)(k.rows == kvq::kF32Rows && m * ratio <= 0x7fffffff ? ratio : 1);
    const int64_t rows = m * sp.pack;
    sp.row_blocks = (int32_t)((rows + k.rows - 1) / k.rows);
    sp.part_blocks = (int32_t)(rows < k.rows ? (rows + 31) / 32 : k.rows / 32);
    const int64_t units = sp.row_blocks * heads * (ratio / sp.pack), rest = units % kComputeUnits;
    auto piece_cost = [&](int64_t s) {
        const int64_t steps = (tiles + s * k.tiles_step - 1) / (s * k.tiles_step);
        return (double)(steps * k.tiles_step) * k.tile + k.fixed;
    };
    auto launchable = [&](int64_t workgroups) { return workgroups * k.threads <= 0xffffffffll; };   // threads of a grid: 32 bits
    if (!launchable(units)) return Plan{sp, kTooLarge};
    int64_t best = 1;
    double best_cost = rest > 0 ? piece_cost(1) : 0.0;
    for (int64_t s = 2; may_split && rest > 0 && s <= kMaxSplits && s <= tiles && rest * s <= kvq::kMaxPieces; ++s) {
        const int64_t rounds = (rest * s + kComputeUnits - 1) / kComputeUnits;
        const double cost = (double)rounds * piece_cost(s) + k.merge + kMergePerSplit * (double)s +
                            kMergePerBlock * (double)(rest * s * sp.part_blocks);
        if (cost < best_cost && launchable(units - rest + rest * s)) {
            best_cost = cost;
            best = s;
        }
    }
    // A split has to promise something: the estimate leaves out that a chip with idle compute units clocks higher, and
    // that pieces of one unit compete for the same memory (31 heads x 1763 rows x 44075 keys, 217 units: 1319 us whole, 1393
    // us in 7 pieces, estimated 1401 and 1351).
    if (best > 1 && best_cost > 0.85 * piece_cost(1)) {
        best = 1;
        best_cost = piece_cost(1);
    }
    sp.splits = (int32_t)best;
    sp.pieces = (int32_t)(best > 1 ? rest * best : 0);
    sp.whole = (int32_t)(best > 1 ? units - rest : units);
    return Plan{sp, best_cost + (double)(units / kComputeUnits) * piece_cost(1)};
}

enum class Route { vector, per_token, group, f32 };

// The kernel that serves a cache's calls, unless the call itself asks for the vector kernel: 16-bit matrix cores for BF16
// and head_dim 128, fp32 matrix cores for the other per-token caches.
Route route_of(const kvq_cache_desc &d, const kvq::CacheView &cv)
{
    if (kvq::attention_mfma_group_supported(cv)) return Route::group;
    if (d.io_dtype == KVQ_BF16 && d.head_dim == 128 && d.group_size == d.head_dim) return Route::per_token;
    return d.key_axis == KVQ_KEYS_PER_TOKEN ? Route::f32 : Route::vector;
}
const KernelCost &cost_of(Route r, int head_dim)
{
    if (r == Route::f32) return head_dim == 64 ? kCostF32Dim64 : kCostF32Dim128;
    return r == Route::group ? kCostGroup : kCostPerToken;
}

// Kernel and grid of a call.  The fp32 kernel's units are 32 rows over all query heads of a key/value head and its tile costs a
// third of a 16-bit kernel's, which however works for eight times the rows: it is the faster one wherever the 256-row blocks do
// not fill the chip about once (a decoded token, the last tokens of a prompt, one to eight heads over some thousand rows).  8
// key/value heads with 4 query heads each, 1 row, 8192 + 64 keys, groups of 32: 70 us in the group-wise kernel, 21 us here; 8
// heads x 143 rows x 286 keys: 31 and 13 us; 16 x 8 heads x 19 rows x 13314 keys, 128 blocks of 256 rows: 524 and 174 us.  Where
// the line lies: 800 random calls of these caches, 1 to 48 heads, 1 to 5000 rows, up to 60000 keys, keys with and without a large
// channel, a quarter of them without a work space, were timed on both kernels.  Where the estimate promised less than 0.8 the fp32
// kernel took 0.51 of the other's time on average and none of 665 calls was slower by more than 1 %; between 0.8 and 0.95 0.83 (2
// of 42 slower, at most 1.10); from there to 1.25 as long (20 of 43 slower, at most 1.35).
struct Choice {
    Route route;
    kvq::SplitArgs sp;
    bool fits;
};
Choice choose(Route route, const kvq_cache_desc &d, int64_t m, int64_t ratio, int64_t tiles, bool may_split)
{
    const Plan p = plan_split(cost_of(route, d.head_dim), m, d.num_heads, ratio, tiles, may_split);
    if (route != Route::f32 && d.key_axis == KVQ_KEYS_PER_TOKEN) {
        const Plan f = plan_split(cost_of(Route::f32, d.head_dim), m, d.num_heads, ratio, tiles, may_split);
        if (f.cost < 0.8 * p.cost) return Choice{Route::f32, f.sp, true};
    }
    return Choice{route, p.sp, p.cost < kTooLarge};
}

// The appended blocks of a per-channel cache that the window [w0, w1) overlaps, listed for the matrix-core kernel, which walks
// the window block by block.  0: it cannot (no cached keys, or more blocks than the list holds).
int list_key_blocks(const std::deque<kvq_block> &blocks, int64_t w0, int64_t w1, kvq::KeyBlock (&list)[kvq::kMaxKeyBlocks])
{
    int n = 0;
    for (const kvq_block &b : blocks) {
        const int64_t s0 = b.start > w0 ? b.start : w0, s1 = b.start + b.count < w1 ? b.start + b.count : w1;
        if (s0 >= s1) continue;
        if (n == kvq::kMaxKeyBlocks) return 0;
        list[n++] = kvq::KeyBlock{(int32_t)b.slot, (int32_t)(s0 - w0), (int32_t)(s1 - w0)};
    }
    return n;
}
// (the matrix-core loaders do their ring arithmetic and their offsets inside a head in 32 bits)
bool beyond_matrix_loaders(const kvq::CacheView &cv, int64_t cache_len)
{
    return cache_len >= (int64_t(1) << 31) || cv.cap_tiles >= (int64_t(1) << 20);
}

// Tiles of a call's key range: cached tiles that the window touches and tiles of the current block.
int64_t key_tiles(int64_t start, int64_t cache_len, int64_t n_cur)
{
    const int64_t cached = cache_len > 0 ? (start + cache_len - 1) / kvq::kTileTokens - start / kvq::kTileTokens + 1 : 0;
    return cached + (n_cur + kvq::kTileTokens - 1) / kvq::kTileTokens;
}

}  // namespace

extern "C" {

size_t kvq_cache_bytes(const kvq_cache_desc *desc)
{
    if (check_desc(desc) != KVQ_OK) return 0;
    const int64_t cap32 = round_up_tile(desc->capacity_tokens);
    const int64_t meta = desc->meta_format == KVQ_META_FP32 ? 8 : 3 * (desc->head_dim / desc->group_size);
    const int64_t per_token = desc->head_dim * desc->bits / 8 + meta;
    return (size_t)(2 * (int64_t)desc->num_heads * cap32 * per_token + channel_bytes(desc, cap32) + kvq::kStatusBytes);
}

kvq_status kvq_cache_create(const kvq_cache_desc *desc, void *dev_mem, size_t bytes, kvq_cache **out)
{
    if (!out) return KVQ_ERR_INVALID_ARG;
    *out = nullptr;
    const kvq_status st = check_desc(desc);
    if (st != KVQ_OK) return st;
    if (!dev_mem || reinterpret_cast<uintptr_t>(dev_mem) % 256 != 0) return KVQ_ERR_INVALID_ARG;
    if (bytes < kvq_cache_bytes(desc)) return KVQ_ERR_INVALID_ARG;
    kvq_cache *c = new (std::nothrow) kvq_cache;
    if (!c) return KVQ_ERR_INVALID_ARG;
    c->desc = *desc;
    c->cap32 = round_up_tile(desc->capacity_tokens);
    c->len = 0;
    c->base = 0;
    c->next_slot = 0;
    c->status_clean = false;
    const int64_t H = desc->num_heads;
    const int64_t code_bytes = H * c->cap32 * desc->head_dim * desc->bits / 8;  // multiple of 256
    const int64_t meta_bytes = H * c->cap32 * 4;                                // multiple of 128
    char *p = static_cast<char *>(dev_mem);
    kvq::CacheView &v = c->view;
    v.k_codes = reinterpret_cast<uint32_t *>(p); p += code_bytes;
    v.v_codes = reinterpret_cast<uint32_t *>(p); p += code_bytes;
    v.k_scale = v.k_negzero = v.v_scale = v.v_zero_off = nullptr;
    v.k_scale8 = v.v_scale8 = nullptr;
    v.k_zero16 = v.v_zero16 = nullptr;
    v.group_size = desc->group_size;
    v.meta_format = desc->meta_format;
    if (desc->meta_format == KVQ_META_FP32) {
        v.k_scale = reinterpret_cast<float *>(p); p += meta_bytes;
        v.k_negzero = reinterpret_cast<float *>(p); p += meta_bytes;
        v.v_scale = reinterpret_cast<float *>(p); p += meta_bytes;
        v.v_zero_off = reinterpret_cast<float *>(p);
    } else {
        const int64_t groups = H * c->cap32 * (desc->head_dim / desc->group_size);   // multiple of 32
        v.k_zero16 = reinterpret_cast<uint16_t *>(p); p += 2 * groups;
        v.v_zero16 = reinterpret_cast<uint16_t *>(p); p += 2 * groups;
        v.k_scale8 = reinterpret_cast<uint8_t *>(p); p += groups;
        v.v_scale8 = reinterpret_cast<uint8_t *>(p); p += groups;
    }
    v.key_axis = desc->key_axis;
    v.max_blocks = 0;
    v.kc_scale = v.kc_zero = nullptr;
    v.k_block = nullptr;
    v.kc_range = nullptr;
    if (desc->key_axis == KVQ_KEYS_PER_CHANNEL) {
        // p stands after the four fp32 arrays of KVQ_META_FP32: a multiple of 128 bytes from a 256-byte base
        p = static_cast<char *>(dev_mem) + 2 * code_bytes + 4 * meta_bytes;
        const int64_t hd = H * desc->head_dim;
        v.max_blocks = (int32_t)max_blocks_of(c->cap32);
        v.kc_range = reinterpret_cast<unsigned long long *>(p); p += hd * 16;   // 8-byte types first
        p += hd * 16;   // (not used: keeps the size and the order of the storage)
        v.kc_scale = reinterpret_cast<float *>(p); p += (int64_t)v.max_blocks * hd * 4;
        v.kc_zero = reinterpret_cast<float *>(p); p += (int64_t)v.max_blocks * hd * 4;
        v.k_block = reinterpret_cast<uint32_t *>(p);
    }
    // every part before it is a multiple of 128 bytes: the status block is 4-byte aligned (it holds 32-bit words)
    v.status = reinterpret_cast<uint32_t *>(static_cast<char *>(dev_mem) + kvq_cache_bytes(desc) - kvq::kStatusBytes);
    v.cap_tiles = c->cap32 / kvq::kTileTokens;
    v.num_heads = desc->num_heads;
    v.head_dim = desc->head_dim;
    v.bits = desc->bits;
    v.io_dtype = desc->io_dtype;
    for (uint32_t &w : v.sign_mask) w = 0u;
    *out = c;
    return KVQ_OK;
}

void kvq_cache_destroy(kvq_cache *cache) { delete cache; }

int64_t kvq_cache_len(const kvq_cache *cache) { return cache ? cache->len : -1; }

kvq_status kvq_cache_reset(kvq_cache *cache)
{
    if (!cache) return KVQ_ERR_INVALID_ARG;
    cache->len = 0;
    cache->base = 0;
    cache->blocks.clear();
    cache->status_clean = false;   // the next append clears the sticky flag before it writes
    return KVQ_OK;
}

kvq_status kvq_cache_set_rotation_signs(kvq_cache *cache, const uint8_t *negate)
{
    if (!cache) return KVQ_ERR_INVALID_ARG;
    if (cache->len != 0) return KVQ_ERR_INVALID_ARG;   // codes already stored belong to the old rotation
    for (uint32_t &w : cache->view.sign_mask) w = 0u;
    if (negate)
        for (int c = 0; c < cache->desc.head_dim; ++c)
            if (negate[c]) cache->view.sign_mask[c >> 5] |= 1u << (c & 31);
    return KVQ_OK;
}

kvq_status kvq_cache_evict(kvq_cache *cache, int64_t n_tokens)
{
    if (!cache || n_tokens < 0 || n_tokens > cache->len) return KVQ_ERR_INVALID_ARG;
    cache->base += n_tokens;
    cache->len -= n_tokens;
    if (cache->len == 0) cache->base = 0;   // an empty cache starts over at a tile boundary
    cache->trim_blocks();
    return KVQ_OK;
}

kvq_status kvq_cache_truncate(kvq_cache *cache, int64_t new_len)
{
    if (!cache || new_len < 0 || new_len > cache->len) return KVQ_ERR_INVALID_ARG;
    cache->len = new_len;
    cache->trim_blocks();
    return KVQ_OK;
}

static kvq_status quantize_append_common(kvq_cache *cache, const void *k, const void *v, int64_t n_tokens,
                                         int64_t stride_token, int64_t stride_head, void *hip_stream, bool static_scratch)
{
    if (!cache || n_tokens < 0) return KVQ_ERR_INVALID_ARG;
    if (static_scratch && (int64_t)cache->desc.num_heads * cache->desc.head_dim > kvq::kStaticScratchChannels)
        return KVQ_ERR_CAPACITY;
    if (n_tokens == 0) return KVQ_OK;
    const kvq_cache_desc &d = cache->desc;
    if (!tensor_ok(k, stride_token, stride_head, d.head_dim, d.io_dtype) ||
        !tensor_ok(v, stride_token, stride_head, d.head_dim, d.io_dtype))
        return KVQ_ERR_INVALID_ARG;
    if (n_tokens > d.capacity_tokens - cache->len) return KVQ_ERR_CAPACITY;
    // Ring storage: the tiles touched by the live tokens and the new ones must all be distinct.
    const int64_t first_tile = cache->base / kvq::kTileTokens;
    const int64_t last_tile = (cache->base + cache->len + n_tokens - 1) / kvq::kTileTokens;
    if (last_tile - first_tile + 1 > cache->view.cap_tiles) return KVQ_ERR_CAPACITY;
    int slot = 0;
    if (d.key_axis == KVQ_KEYS_PER_CHANNEL) {
        if ((int64_t)cache->blocks.size() >= cache->view.max_blocks) return KVQ_ERR_CAPACITY;
        slot = cache->next_slot;
    }
    if (!cache->status_clean) {
        if (kvq::launch_status_clear(cache->view, static_cast<hipStream_t>(hip_stream)) != hipSuccess) return KVQ_ERR_HIP;
        cache->status_clean = true;
    }
    const hipError_t e = kvq::launch_quantize_append(cache->view, k, v, cache->base + cache->len, n_tokens, stride_token,
                                                     stride_head, slot, static_cast<hipStream_t>(hip_stream), static_scratch);
    if (e != hipSuccess) return KVQ_ERR_HIP;
    if (d.key_axis == KVQ_KEYS_PER_CHANNEL) {
        cache->blocks.push_back(kvq_block{slot, cache->base + cache->len, n_tokens});
        cache->next_slot = (slot + 1) % cache->view.max_blocks;
    }
    cache->len += n_tokens;
    return KVQ_OK;
}

kvq_status kvq_quantize_append(kvq_cache *cache, const void *k, const void *v, int64_t n_tokens,
                               int64_t stride_token, int64_t stride_head, void *hip_stream)
{
    return quantize_append_common(cache, k, v, n_tokens, stride_token, stride_head, hip_stream, false);
}

kvq_status kvq_quantize_append_static(kvq_cache *cache, const void *k, const void *v, int64_t n_tokens,
                                      int64_t stride_token, int64_t stride_head, void *hip_stream)
{
    return quantize_append_common(cache, k, v, n_tokens, stride_token, stride_head, hip_stream, true);
}

static kvq_status attention_common(const kvq_cache *cache, int64_t cache_start, int64_t cache_len,
                                   const void *q, const void *k_cur, const void *v_cur, int64_t m,
                                   int64_t n_cur, int64_t stride_token, int64_t stride_head,
                                   float softmax_scale, int correction, void *out, float *mass_cached,
                                   void *hip_stream, bool force_vector, const kvq_attention_opts *opts = nullptr,
                                   const void *k_ref = nullptr, const void *v_ref = nullptr, float *diag = nullptr,
                                   void *workspace = nullptr, size_t workspace_bytes = 0)
{
    // diag != nullptr: the diagnostics call (no out / mass_cached; k_ref, v_ref hold the cached tokens unquantized)
    kvq_attention_opts o = {1, 0, stride_token, stride_head};
    if (opts) {
        o = *opts;
        if (o.q_stride_token == 0 && o.q_stride_head == 0) {
            o.q_stride_token = stride_token;
            o.q_stride_head = stride_head;
        }
        if (o.q_heads_per_kv_head < 1 || o.q_heads_per_kv_head > 64) return KVQ_ERR_INVALID_ARG;
        if (o.causal != 0 && o.causal != 1) return KVQ_ERR_INVALID_ARG;
        if (o.causal && n_cur < m) return KVQ_ERR_INVALID_ARG;   // the queries are the last m current positions
    }
    if (!cache || m < 0 || n_cur < 0 || cache_len < 0 || cache_start < 0) return KVQ_ERR_INVALID_ARG;
    if (cache_start + cache_len > cache->len) return KVQ_ERR_INVALID_ARG;
    if (cache_len == 0 && n_cur == 0) return KVQ_ERR_INVALID_ARG;
    if (correction < 0 || correction > 2) return KVQ_ERR_INVALID_ARG;
    if (!(softmax_scale >= 0.0f) || !(softmax_scale < 3.0e38f)) return KVQ_ERR_INVALID_ARG;
    if (m == 0) return KVQ_OK;
    const kvq_cache_desc &d = cache->desc;
    if (!tensor_ok(q, o.q_stride_token, o.q_stride_head, d.head_dim, d.io_dtype)) return KVQ_ERR_INVALID_ARG;
    if (!diag && !tensor_ok(out, o.q_stride_token, o.q_stride_head, d.head_dim, d.io_dtype)) return KVQ_ERR_INVALID_ARG;
    if (diag && cache_len > 0 && (!tensor_ok(k_ref, stride_token, stride_head, d.head_dim, d.io_dtype) ||
                                  !tensor_ok(v_ref, stride_token, stride_head, d.head_dim, d.io_dtype)))
        return KVQ_ERR_INVALID_ARG;
    if (diag && reinterpret_cast<uintptr_t>(diag) % 4 != 0) return KVQ_ERR_INVALID_ARG;
    if (n_cur > 0 && (!tensor_ok(k_cur, stride_token, stride_head, d.head_dim, d.io_dtype) ||
                      !tensor_ok(v_cur, stride_token, stride_head, d.head_dim, d.io_dtype)))
        return KVQ_ERR_INVALID_ARG;
    if (mass_cached && reinterpret_cast<uintptr_t>(mass_cached) % 4 != 0) return KVQ_ERR_INVALID_ARG;
    if (!diag && (out == q || out == k_cur || out == v_cur)) return KVQ_ERR_INVALID_ARG;
    if (m > ((int64_t)1 << 31) - 256 || n_cur > ((int64_t)1 << 31) - 256) return KVQ_ERR_INVALID_ARG;

    kvq::AttentionArgs a;
    a.cv = cache->view;
    a.cache_start = cache->base + cache_start;
    a.cache_len = cache_len;
    a.phys_tile_first = (a.cache_start / kvq::kTileTokens) % cache->view.cap_tiles;
    a.q = q;
    a.k_cur = k_cur;
    a.v_cur = v_cur;
    a.m = m;
    a.n_cur = n_cur;
    a.stride_token = stride_token;
    a.stride_head = stride_head;
    a.q_stride_token = o.q_stride_token;
    a.q_stride_head = o.q_stride_head;
    a.q_per_kv = o.q_heads_per_kv_head;
    a.causal = o.causal;
    a.softmax_scale = softmax_scale > 0.0f ? softmax_scale : (d.head_dim == 64 ? 0.125f : 0.088388347648318f);
    a.correction = correction;
    a.out = out;
    a.mass_cached = mass_cached;
    a.n_key_blocks = 0;
    a.status = cache->status_clean && cache_len > 0 ? cache->view.status : nullptr;
    a.only_if_flagged = 0;
    // the exact (sinh) correction is a diagnostic mode: vector kernel only
    force_vector = force_vector || correction == 2;
    if (d.key_axis == KVQ_KEYS_PER_CHANNEL && !force_vector) {
        a.n_key_blocks = list_key_blocks(cache->blocks, a.cache_start, a.cache_start + cache_len, a.key_blocks);
        force_vector = a.n_key_blocks == 0;
    }
    force_vector = force_vector || beyond_matrix_loaders(cache->view, cache_len);
    const hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (diag) return kvq::launch_diagnostics_simt(a, k_ref, v_ref, diag, s) == hipSuccess ? KVQ_OK : KVQ_ERR_HIP;
    const Route own = force_vector ? Route::vector : route_of(d, cache->view);
    if (own == Route::vector) return kvq::launch_attention_simt(a, s) == hipSuccess ? KVQ_OK : KVQ_ERR_HIP;
    const int64_t ratio = o.q_heads_per_kv_head, tiles = key_tiles(a.cache_start, cache_len, n_cur);
    Choice c = choose(own, d, m, ratio, tiles, true);
    if (workspace_bytes < kvq::split_workspace_bytes(c.sp, d.head_dim)) c = choose(own, d, m, ratio, tiles, false);
    if (!c.fits && c.route == Route::f32) return kvq::launch_attention_simt(a, s) == hipSuccess ? KVQ_OK : KVQ_ERR_HIP;
    if (!c.fits) return KVQ_ERR_HIP;
    const Route route = c.route;
    kvq::SplitArgs &sp = c.sp;
    sp.part_o = static_cast<float *>(workspace);
    sp.part_ml = reinterpret_cast<float4 *>(sp.part_o + (size_t)sp.pieces * sp.part_blocks * 32 * d.head_dim);
    if (route == Route::f32) a.status = nullptr;   // any zero-point will do
    const bool split = sp.pieces > 0;
    auto launch = route == Route::f32         ? kvq::launch_attention_f32
                  : route == Route::per_token ? (split ? kvq::launch_attention_mfma_split : kvq::launch_attention_mfma)
                                              : (split ? kvq::launch_attention_mfma_group_split : kvq::launch_attention_mfma_group);
    hipError_t e = launch(a, sp, s);
    if (e != hipSuccess) return KVQ_ERR_HIP;
    if (split) {
        e = route == Route::f32 ? kvq::launch_attention_merge(a, sp, s) : kvq::launch_attention_merge_or_vector(a, sp, s);
    } else if (a.status) {
        // A cache that has ever stored a zero-point beyond the 16-bit kernels' domain carries a flag: the launch
        // above has then returned without writing anything, and this one, which otherwise returns at once, does the work.
        a.only_if_flagged = 1;
        e = kvq::launch_attention_simt(a, s);
    }
    return e == hipSuccess ? KVQ_OK : KVQ_ERR_HIP;
}

kvq_status kvq_chunk_attention(const kvq_cache *cache, int64_t cache_start, int64_t cache_len,
                               const void *q, const void *k_cur, const void *v_cur, int64_t m,
                               int64_t n_cur, int64_t stride_token, int64_t stride_head,
                               float softmax_scale, int correction, void *out, float *mass_cached,
                               void *hip_stream)
{
    return attention_common(cache, cache_start, cache_len, q, k_cur, v_cur, m, n_cur, stride_token, stride_head,
                            softmax_scale, correction, out, mass_cached, hip_stream, false);
}

kvq_status kvq_chunk_attention_fp32(const kvq_cache *cache, int64_t cache_start, int64_t cache_len,
                                    const void *q, const void *k_cur, const void *v_cur, int64_t m,
                                    int64_t n_cur, int64_t stride_token, int64_t stride_head,
                                    float softmax_scale, int correction, void *out, float *mass_cached,
                                    void *hip_stream)
{
    return attention_common(cache, cache_start, cache_len, q, k_cur, v_cur, m, n_cur, stride_token, stride_head,
                            softmax_scale, correction, out, mass_cached, hip_stream, true);
}

kvq_status kvq_chunk_attention_ex(const kvq_cache *cache, int64_t cache_start, int64_t cache_len,
                                  const void *q, const void *k_cur, const void *v_cur, int64_t m,
                                  int64_t n_cur, int64_t stride_token, int64_t stride_head,
                                  float softmax_scale, int correction, const kvq_attention_opts *opts,
                                  void *out, float *mass_cached, void *hip_stream)
{
    return attention_common(cache, cache_start, cache_len, q, k_cur, v_cur, m, n_cur, stride_token, stride_head,
                            softmax_scale, correction, out, mass_cached, hip_stream, false, opts);
}

size_t kvq_attention_workspace_bytes(const kvq_cache *cache, int64_t cache_start, int64_t cache_len, int64_t m, int64_t n_cur,
                                     int q_heads_per_kv_head)
{
    if (!cache || m <= 0 || n_cur < 0 || cache_len < 0 || cache_start < 0 || q_heads_per_kv_head < 1 || q_heads_per_kv_head > 64) return 0;
    const kvq_cache_desc &d = cache->desc;
    const Route route = route_of(d, cache->view);
    if (route == Route::vector || cache_len > cache->len - cache_start || beyond_matrix_loaders(cache->view, cache_len)) return 0;
    if (m > ((int64_t)1 << 31) - 256 || n_cur > ((int64_t)1 << 31) - 256) return 0;
    const int64_t start = cache->base + cache_start, tiles = key_tiles(start, cache_len, n_cur);
    kvq::KeyBlock list[kvq::kMaxKeyBlocks];
    if (d.key_axis == KVQ_KEYS_PER_CHANNEL && list_key_blocks(cache->blocks, start, start + cache_len, list) == 0) return 0;
    return kvq::split_workspace_bytes(choose(route, d, m, q_heads_per_kv_head, tiles, true).sp, d.head_dim);
}

kvq_status kvq_chunk_attention_ws(const kvq_cache *cache, int64_t cache_start, int64_t cache_len,
                                  const void *q, const void *k_cur, const void *v_cur, int64_t m,
                                  int64_t n_cur, int64_t stride_token, int64_t stride_head,
                                  float softmax_scale, int correction, const kvq_attention_opts *opts,
                                  void *out, float *mass_cached, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (workspace ? reinterpret_cast<uintptr_t>(workspace) % 256 != 0 : workspace_bytes != 0) return KVQ_ERR_INVALID_ARG;
    return attention_common(cache, cache_start, cache_len, q, k_cur, v_cur, m, n_cur, stride_token, stride_head,
                            softmax_scale, correction, out, mass_cached, hip_stream, false, opts, nullptr, nullptr, nullptr,
                            workspace, workspace_bytes);
}

kvq_status kvq_attention_diagnostics(const kvq_cache *cache, int64_t cache_start, int64_t cache_len, const void *q,
                                     const void *k_ref, const void *v_ref, const void *k_cur, const void *v_cur,
                                     int64_t m, int64_t n_cur, int64_t stride_token, int64_t stride_head,
                                     float softmax_scale, int correction, float *diag, void *hip_stream)
{
    if (!diag) return KVQ_ERR_INVALID_ARG;
    return attention_common(cache, cache_start, cache_len, q, k_cur, v_cur, m, n_cur, stride_token, stride_head,
                            softmax_scale, correction, nullptr, nullptr, hip_stream, true, nullptr, k_ref, v_ref, diag);
}

kvq_status kvq_cache_export(const kvq_cache *cache, int which, int64_t start, int64_t count, uint8_t *codes,
                            float *scales, float *zeros, void *hip_stream)
{
    if (!cache || (which != 0 && which != 1) || start < 0 || count < 0) return KVQ_ERR_INVALID_ARG;
    if (start + count > cache->len) return KVQ_ERR_INVALID_ARG;
    if (count == 0) return KVQ_OK;
    const hipError_t e = kvq::launch_export(cache->view, which, cache->base + start, count, codes, scales, zeros,
                                            static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? KVQ_OK : KVQ_ERR_HIP;
}

const char *kvq_status_string(kvq_status status)
{
    switch (status) {
        case KVQ_OK: return "ok";
        case KVQ_ERR_INVALID_ARG: return "invalid argument";
        case KVQ_ERR_UNSUPPORTED: return "unsupported configuration";
        case KVQ_ERR_CAPACITY: return "cache capacity exceeded";
        case KVQ_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

const char *kvq_version(void) { return "0.2"; }

}  // extern "C"
