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

// Lists the same items in the same places, for batches of so many that finding each when it is due costs more than a kernel in front: a
// wavefront finds the tile at a position, for all heads at once, and writes its items.  Chains of trips to memory and of cross-lane
// sums are what it takes, so every position has its own wavefront; no wavefront waits for another.  24 to 256 sequences, 16 and 8 heads: 6.2 us on average,
// where one workgroup (build_static_queue_kernel) took 9.5 (profiler on).
__global__ __launch_bounds__(kThreads) void list_items_kernel(const AttnArgs)
{
    KernArgs &a = kernel_args();
    const int lane = thread_id() & 63;
    const int first = workgroup_id() * (kThreads / 64) + __builtin_amdgcn_readfirstlane(thread_id() >> 6), waves = a.grid * (kThreads / 64);
    for (int i = first * 64 + lane; i < kStaticRecords; i += waves * 64) a.pq.split_flags[i] = 0;
    const SearchBatch<kSearchSeqs / 64> batch(a, lane);
    const int total = batch.total, nq = kMaxQueues, heads = a.Hq;
    auto queue_start = [&](int x) { return x * (total / nq) + min(x, total % nq); };
    if (first == 0 && lane <= nq) {
        ((int32_t *)a.pq.offsets)[lane] = queue_start(lane);
        a.pq.counters[lane * kCounterStride] = 0;
    }
    flexsp_item *const items = (flexsp_item *)a.pq.items;
    for (int pos = first; pos < total / heads; pos += waves) {
        const flexsp_item it = batch.tile(a, pos, lane);
        for (int h = lane; h < heads; h += 64) {
            const int2 at = batch.queue_place(heads, pos, h);
            items[queue_start(at.x) + at.y] = batch.head_of(it, h);
        }
    }
}

}  // namespace

hipError_t launch_list_items(const AttnArgs &a, int positions, hipStream_t s)
{
    launch(list_items_kernel, a, (positions + kThreads / 64 - 1) / (kThreads / 64), s);
    return hipGetLastError();
}

hipError_t launch_attn_fwd_search(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    launch(D == 128 ? attn_fwd_search_kernel<128> : attn_fwd_search_kernel<64>, a, grid, s);
    return hipGetLastError();
}

}  // namespace flexsp
