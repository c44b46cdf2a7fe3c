// The merge kernel of the fp32 matrix-core launches (the 16-bit ones are merged by attention_merge_or_vector_kernel).
#include "kvq_internal.h"

namespace kvq {
namespace {
#include "kvq_merge.h"

template <int DIM, typename T> __global__ __launch_bounds__(kMergeThreads) void attention_merge_kernel(AttentionArgs a, SplitArgs sp)
{
    merge_rows<DIM, T, false>(a, sp);
}

}  // namespace

template <int DIM, typename T> static hipError_t launch_merge(const AttentionArgs &a, const SplitArgs &sp, hipStream_t stream)
{
    return launch_kernel(attention_merge_kernel<DIM, T>, dim3(merge_workgroups<DIM>(sp)), dim3(kMergeThreads), 0, stream, a, sp);
}
hipError_t launch_attention_merge(const AttentionArgs &a, const SplitArgs &sp, hipStream_t stream)
{
    const bool bf16 = a.cv.io_dtype == KVQ_BF16;
    if (a.cv.head_dim == 128) return bf16 ? launch_merge<128, uint16_t>(a, sp, stream) : launch_merge<128, float>(a, sp, stream);
    return bf16 ? launch_merge<64, uint16_t>(a, sp, stream) : launch_merge<64, float>(a, sp, stream);
}

}  // namespace kvq
