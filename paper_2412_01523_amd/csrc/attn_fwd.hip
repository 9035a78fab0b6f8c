// The forward's kernels: with a list of items, without one for batches of few items, for key shards, and in halves.
#include "attn_fwd_search.h"

namespace flexsp {
namespace {

template <int D, bool SHARD, bool FIND, int HALVES>
__global__ __launch_bounds__(kThreads, HALVES == 2 ? 1 : D == 64 && !SHARD ? 3 : 2) void attn_fwd_kernel(const AttnArgs)
{
    __shared__ __attribute__((aligned(1024))) char smem[fwd_lds<D, HALVES, 2>()];
    __shared__ __attribute__((aligned(8))) float stats[fwd_stats<HALVES>()];
    __shared__ int deal_word, split_word;
    KernArgs &args = kernel_args();
    flexsp_item found;
    if constexpr (FIND) {
        if (!find_item(args.cu, args.B, args.T, args.Hq, args.causal, workgroup_id(), thread_id() & 63, found)) return;
    }
    fwd_pass<D, SHARD, FIND, HALVES>(args, found, smem, stats, deal_word, split_word);
}

// The forward without a plan where only the lengths on the device tell whether the batch runs in halves: the host knows the rows that the
// tensors hold, and the batch may be shorter.  Either kind of items is found in the lengths; BUFS = 2 is for launches of so few items that a
// compute unit's LDS is theirs, DEAL = true for launches of more whole items than workgroups.
template <int D, int BUFS, bool DEAL>
__global__ __launch_bounds__(kThreads, D == 128 && BUFS == 2 ? 1 : 2) void attn_fwd_either_kernel(const AttnArgs)
{
    __shared__ __attribute__((aligned(1024))) char smem[fwd_lds<D, 2, BUFS>()];
    static_assert(fwd_lds<D, 2, BUFS>() >= fwd_lds<D, 1, 2>(), "LDS of either pass");
    __shared__ __attribute__((aligned(8))) float stats[fwd_stats<2>()];
    __shared__ int deal_word, split_word;
    KernArgs &args = kernel_args();
    flexsp_item found;
    if constexpr (DEAL) {
        // (the lengths are looked at again for every item: kept, they would be registers that the passes do not have)
        if (ShortBatch<D>(fresh(args), thread_id() & 63).halves) {
            for (int n = workgroup_id();; n += args.grid) {
                int lane = thread_id() & 63;
                asm volatile("" : "+v"(lane));
                if (!ShortBatch<D>(fresh(args), lane).item(fresh(args), n, found)) break;
                __syncthreads();  // (everybody is done with the LDS of the one before)
                fwd_pass<D, false, true, 2, BUFS>(args, found, smem, stats, deal_word, split_word);
            }
        } else {
            fwd_pass<D, false, false, 1, 2>(args, found, smem, stats, deal_word, split_word, SearchBatch<1>(args, thread_id() & 63));
        }
        return;
    }
    const ShortBatch<D> batch(args, thread_id() & 63);
    if (batch.halves) {
        for (int n = workgroup_id(); batch.item(args, n, found); n += args.grid) {
            __syncthreads();  // (everybody is done with the LDS of the one before)
            fwd_pass<D, false, true, 2, BUFS>(args, found, smem, stats, deal_word, split_word);
        }
    } else if (batch.item(args, workgroup_id(), found)) {
        fwd_pass<D, false, true, 1>(args, found, smem, stats, deal_word, split_word);
    }
}

}  // namespace

hipError_t launch_attn_fwd(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    if (a.halves && !a.cu)
        launch(D == 128 ? attn_fwd_kernel<128, false, false, 2> : attn_fwd_kernel<64, false, false, 2>, a, grid, s);
    else if (a.halves && a.pq.counters)
        launch(D == 128 ? attn_fwd_either_kernel<128, 1, true> : attn_fwd_either_kernel<64, 1, true>, a, grid, s);
    else if (a.halves)
        launch(D == 64 ? attn_fwd_either_kernel<64, 2, false> : a.halves == 2 ? attn_fwd_either_kernel<128, 2, false> : attn_fwd_either_kernel<128, 1, false>, a, grid, s);
    else if (a.cu)
        launch(D == 128 ? attn_fwd_kernel<128, false, true, 1> : attn_fwd_kernel<64, false, true, 1>, a, grid, s);
    else
        launch(D == 128 ? attn_fwd_kernel<128, false, false, 1> : attn_fwd_kernel<64, false, false, 1>, a, grid, s);
    return hipGetLastError();
}

hipError_t launch_attn_fwd_kvshard(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    launch(D == 128 ? attn_fwd_kernel<128, true, false, 1> : attn_fwd_kernel<64, true, false, 1>, a, grid, s);
    return hipGetLastError();
}

}  // namespace flexsp
