// The merge kernel of the fp32 matrix-core launches (the 16-bit ones are merged by attention_merge_or_vector_kernel).
#include "kvq_internal.h"

namespace kvq {
namespace {
#include "kvq_merge.h"

template <int DIM, typename T> __global__ __launch_bounds__(kMergeThreads) void attention_merge_kernel(AttentionArgs a, SplitArgs sp)
{
    merge_rows<DIM, T>(a, sp);
}

}  // namespace

hipError_t launch_attention_merge(const AttentionArgs &a, const SplitArgs &sp, hipStream_t stream)
{
    const dim3 grid = merge_grid(a, sp);
    const bool bf16 = a.cv.io_dtype == KVQ_BF16;
    if (a.cv.head_dim == 128 && bf16) return launch_kernel(attention_merge_kernel<128, uint16_t>, grid, dim3(kMergeThreads), 0, stream, a, sp);
    if (a.cv.head_dim == 128) return launch_kernel(attention_merge_kernel<128, float>, grid, dim3(kMergeThreads), 0, stream, a, sp);
    if (bf16) return launch_kernel(attention_merge_kernel<64, uint16_t>, grid, dim3(kMergeThreads), 0, stream, a, sp);
    return launch_kernel(attention_merge_kernel<64, float>, grid, dim3(kMergeThreads), 0, stream, a, sp);
}

}  // namespace kvq
