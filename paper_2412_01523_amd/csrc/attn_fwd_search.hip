// The forward without a plan, for batches of more items than can be resident: its workgroups find the items in the lengths.
#include "attn_fwd_search.h"

namespace flexsp {
namespace {

template <int D>
__global__ __launch_bounds__(kThreads, 2) void attn_fwd_search_kernel(const AttnArgs)
{
    __shared__ __attribute__((aligned(1024))) char smem[fwd_lds<D, 1, 2>()];
    __shared__ __attribute__((aligned(8))) float stats[fwd_stats<1>()];
    __shared__ int deal_word, split_word;
    KernArgs &args = kernel_args();
    const SearchBatch<kSearchSeqs / 64> batch(args, thread_id() & 63);
    fwd_pass<D, false, false, 1, 2>(args, flexsp_item(), smem, stats, deal_word, split_word, batch);
}

}  // namespace

hipError_t launch_attn_fwd_search(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    launch(D == 128 ? attn_fwd_search_kernel<128> : attn_fwd_search_kernel<64>, a, grid, s);
    return hipGetLastError();
}

}  // namespace flexsp
