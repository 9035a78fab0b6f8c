// Host side of libflexsp: contexts, tile plans, argument validation and the extern "C"
// entry points declared in include/flexsp.h.  No kernel lives here.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "flexsp_internal.h"

using namespace flexsp;

struct EventPair {
    hipEvent_t start, stop;
    int kernel;
};

// Device memory of a plan plus the pinned host buffer its queues are uploaded from.  Slabs are
// recycled through the context: creating a plan per micro-batch then costs neither an allocation
// nor a device-wide synchronisation (hipFree), and the upload is an asynchronous copy.
struct PlanSlab {
    void *dev = nullptr;
    size_t dev_bytes = 0;
    void *host = nullptr;  // pinned
    size_t host_bytes = 0;
    hipEvent_t ready = nullptr;  // recorded on the upload stream after the copy
    hipEvent_t done = nullptr;   // recorded on the last stream that ran kernels on this slab
    bool done_valid = false;
};
constexpr size_t kSlabPoolMax = 16;  // free slabs kept by a context
constexpr size_t kSlabEager = 4;     // slabs a context makes rather than wait for a busy one ...
constexpr size_t kSlabEagerBytes = (size_t)8 << 30;  // ... while they hold less device memory than this (a backward in one pass keeps 512 bytes a token and head)
constexpr size_t kSlabPoolBytes = (size_t)16 << 30;  // free slabs hold no more device memory than this, the one released last apart
constexpr size_t kSlabWaste = (size_t)64 << 20;      // a plan takes no slab of more than four times what it asks for and this

struct flexsp_ctx {
    int device;  // -1: host-only
    int num_cu;
    int num_xcd;
    hipStream_t upload = nullptr;  // non-blocking stream (default priority) for plan uploads
    std::vector<PlanSlab> slabs;   // free slabs
    size_t slabs_owned = 0;        // slabs alive: free ones and those held by plans
    size_t slab_bytes = 0;         // device memory of the slabs alive
    // profiling: a pool of event pairs created by flexsp_profile_start
    bool profiling;
    std::vector<EventPair> events;
    size_t events_used;
    int64_t dropped;
};

struct HostPass {
    std::vector<flexsp_item> items;     // queue order
    int64_t offsets[kMaxQueues + 1];    // queue boundaries
    int tile_rows;
    int32_t records = 0;                // partial-result records of split tiles
    int64_t steps = 0, longest = 0;     // inner-loop steps of the pass and of its longest item
    std::vector<flexsp_item> direct;    // items in workgroup order, if the pass is launched with one workgroup per item
};

struct flexsp_plan {
    flexsp_ctx *ctx;
    int32_t B, Hq, Hkv, D, causal;
    int64_t T;
    std::vector<int32_t> cu;
    // key-shard plans (forward only): the shard's own boundaries and the position offsets
    bool kvshard = false;
    std::vector<int32_t> cu_k, shift;
    int64_t Tk = 0;
    bool wide = false;  // the dK/dV pass's items have kDkvWideBk keys
    mutable bool two_listed = true;  // the two backward passes are listed (a plan that runs in one lists them when somebody asks)
    bool halves = false;  // the forward is launched in halves: its direct list has kHalfBq query rows to an item
    mutable HostPass pass[3];
    std::vector<flexsp_item> chain;        // items of the backward in one pass (attn_bwd_chain.hip); empty: it runs in two
    std::vector<int32_t> chain_bundles;    // ... boundaries of its bundles
    int64_t chain_tiles = 0;  // tiles of kDkvBq query rows it keeps partial sums of, over all heads
    PassQueues chain_dq;
    // device side (null for host-only plans): one allocation, carved up
    void *dev_base;
    size_t dev_bytes;
    PlanSlab slab;
    bool uploaded;            // the upload is known to have completed
    bool used, multi_stream;  // kernels were launched on this plan; on more than one stream
    hipStream_t last_stream;
    PassQueues dq[3];
    float *delta;
    size_t delta_bytes;
};

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return e == hipErrorOutOfMemory ? FLEXSP_OUT_OF_MEMORY : FLEXSP_HIP_ERROR;
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Workgroups an attention launch keeps resident: two per compute unit (a host-only context plans
// for the 256 compute units of the device it stands in for).
int workgroups_of(const flexsp_ctx *ctx) { return 2 * (ctx->num_cu > 0 ? ctx->num_cu : 256); }

void slab_free(PlanSlab &s)
{
    if (s.dev) (void)hipFree(s.dev);
    if (s.host) (void)hipHostFree(s.host);
    if (s.ready) (void)hipEventDestroy(s.ready);
    if (s.done) (void)hipEventDestroy(s.done);
    s = PlanSlab();
}

// Gives a free slab's memory back, behind its kernels and its upload.
void slab_give_back(flexsp_ctx *ctx, PlanSlab &s)
{
    if (s.done_valid) (void)hipEventSynchronize(s.done);
    (void)hipEventSynchronize(s.ready);
    ctx->slab_bytes -= s.dev_bytes;
    slab_free(s);
    ctx->slabs_owned--;
}

hipError_t slab_make(PlanSlab &s)
{
    hipError_t e = hipMalloc(&s.dev, s.dev_bytes);
    if (e == hipSuccess) e = hipHostMalloc(&s.host, s.host_bytes, hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s.ready, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s.done, hipEventDisableTiming);
    if (e != hipSuccess) {
        const size_t dev_bytes = s.dev_bytes, host_bytes = s.host_bytes;
        slab_free(s);
        s.dev_bytes = dev_bytes;
        s.host_bytes = host_bytes;
    }
    return e;
}

// A slab with at least the given sizes.  Among the adequate ones in the pool, one whose last
// kernels have already finished is preferred (the smallest such): its queues can be uploaded at
// once, while the kernels of the plan destroyed a moment ago still run.  Taking back the slab just
// released instead would put every step's upload behind the previous step's last kernel and in
// front of its own first one, an idle gap per step.  When every adequate slab is still in use
// and the context owns fewer than kSlabEager slabs (and less than kSlabEagerBytes in them), a new one
// is made (a quarter larger than asked, so that the next, slightly different batch fits too).
// Beyond that the HOST waits here for the busy slab released longest ago: a caller that builds a
// plan per micro-batch is thereby held kSlabEager steps ahead of the GPU at most, which keeps the
// GPU fed just as well as running ahead without bound does.  Both alternatives were measured and
// stall the GPU for 6-9 ms each time: making slabs as the host runs further ahead (allocating
// device and pinned memory in the middle of a run), and ordering the upload behind the busy
// slab's kernels with an event on the upload stream (the first such cross-stream waits after an
// idle period).  With the host-side wait, allocations end with the first kSlabEager plans of a run
// and no stream ever waits for an event that is not complete yet.
// A slab that is far too large stays in the pool for a plan that needs it: a small plan would hold gigabytes for its life, and the next large one
// would make another.  Where there is no memory for a new one, the free ones are given back first, those whose kernels have finished before others.
hipError_t slab_get(flexsp_ctx *ctx, size_t dev_bytes, size_t host_bytes, PlanSlab &out)
{
    int best = -1, best_busy = -1;
    for (size_t i = 0; i < ctx->slabs.size(); i++) {
        const PlanSlab &s = ctx->slabs[i];
        if (s.dev_bytes < dev_bytes || s.host_bytes < host_bytes || s.dev_bytes > 4 * dev_bytes + kSlabWaste) continue;
        const bool idle = !s.done_valid || hipEventQuery(s.done) == hipSuccess;
        // idle: the smallest adequate one; busy: the first in the list, which was released first
        if (idle) {
            if (best < 0 || s.dev_bytes < ctx->slabs[best].dev_bytes) best = (int)i;
        } else if (best_busy < 0) {
            best_busy = (int)i;
        }
    }
    if (best < 0 && best_busy >= 0 && (ctx->slabs_owned >= kSlabEager || ctx->slab_bytes + dev_bytes > kSlabEagerBytes))
        best = best_busy;
    if (best >= 0) {
        out = ctx->slabs[best];
        ctx->slabs.erase(ctx->slabs.begin() + best);
        if (best == best_busy) {
            hipError_t e = hipEventSynchronize(out.done);
            if (e != hipSuccess) return e;
        }
        out.done_valid = false;  // its kernels are over: nothing to order the upload behind
        // the previous upload from this pinned buffer must be over before the host refills it
        return hipEventSynchronize(out.ready);
    }
    PlanSlab s;
    s.dev_bytes = dev_bytes + dev_bytes / 4 + 256;
    s.host_bytes = host_bytes + host_bytes / 4 + 256;
    hipError_t e = slab_make(s);
    while (e == hipErrorOutOfMemory && !ctx->slabs.empty()) {
        (void)hipGetLastError();
        size_t room = 0, total = 0;
        if (hipMemGetInfo(&room, &total) != hipSuccess) return e;
        for (const PlanSlab &x : ctx->slabs) room += x.dev_bytes;
        if (room < s.dev_bytes) return e;  // in vain (the next, smaller request may find what it needs in the pool)
        size_t i = 0;
        while (i + 1 < ctx->slabs.size() && ctx->slabs[i].done_valid && hipEventQuery(ctx->slabs[i].done) != hipSuccess) i++;
        if (ctx->slabs[i].done_valid && hipEventQuery(ctx->slabs[i].done) != hipSuccess) i = 0;  // none has finished: the one released first
        slab_give_back(ctx, ctx->slabs[i]);
        ctx->slabs.erase(ctx->slabs.begin() + i);
        e = slab_make(s);
    }
    if (e != hipSuccess) return e;
    ctx->slabs_owned++;
    ctx->slab_bytes += s.dev_bytes;
    out = s;
    return hipSuccess;
}

// Called by the hot entry points before they launch on `stream`: the kernels must see the
// uploaded queues.  Once the upload is known to be complete this is one flag test.
hipError_t plan_before_launch(flexsp_plan *plan, hipStream_t stream)
{
    if (!plan->uploaded) {
        hipError_t q = hipEventQuery(plan->slab.ready);
        if (q == hipSuccess) {
            plan->uploaded = true;
        } else if (q == hipErrorNotReady) {
            hipError_t e = hipStreamWaitEvent(stream, plan->slab.ready, 0);
            if (e != hipSuccess) return e;
        } else {
            return q;
        }
    }
    if (plan->used && plan->last_stream != stream) plan->multi_stream = true;
    plan->used = true;
    plan->last_stream = stream;
    return hipSuccess;
}

// Brackets one kernel launch with a pair of events while profiling is on.
struct Timed {
    flexsp_ctx *ctx;
    hipStream_t stream;
    EventPair *ev;
    Timed(flexsp_ctx *c, int kernel, hipStream_t s) : ctx(c), stream(s), ev(nullptr)
    {
        if (!c->profiling) return;
        if (c->events_used >= c->events.size()) {
            c->dropped++;
            return;
        }
        ev = &c->events[c->events_used++];
        ev->kernel = kernel;
        (void)hipEventRecord(ev->start, stream);
    }
    ~Timed()
    {
        if (ev) (void)hipEventRecord(ev->stop, stream);
    }
};

struct Work {
    flexsp_item it;
    int64_t cost;   // inner-loop steps of this item
    int32_t group;  // (sequence, head) group id
    int32_t keep;   // what is kept on one queue: the group, or the parts of one number of its cut tiles
};

void distribute(std::vector<Work> &work, const std::vector<int64_t> &group_cost, int nq, int n_wg, int tile_rows,
                HostPass &out, int spare = 0, int64_t row_bytes = 0, int heads_walked = 1);

// Groups of one cost go round the queues in the order they are listed in: the n-th head listed of a sequence.  Where every queue gets several
// of its heads it gets neighbours, which share their key head's rows in the XCD's L2 if heads are grouped: 262 144 tokens in
// sequences of up to 65 536, 16 heads on 2, forward and backward 151.7 -> 150.3 ms.  (Same bits; nothing changes for the caches with as many
// key heads as heads, nor with no more heads than queues.  The key heads of a shard's dK/dV pass, which share no rows, are listed as they come.)
int nth_head(int n, int heads, int nq) { return heads % nq ? n : n % nq * (heads / nq) + n / nq; }

// Builds one pass: lists the items, spreads whole (sequence, head) groups over the queues
// (largest group first onto the least loaded queue, so tiles that read the same K/V run on
// one XCD and share its L2), then orders each queue by decreasing cost (short sequences: tile beside tile, see distribute) so that the long
// tail of a batch starts first and short items fill the gaps at the end.
void build_pass(const std::vector<int32_t> &cu, int B, int heads, int group_mult, int tile_rows,
                int step_rows, bool causal, bool key_major, int D, int nq, int n_wg, HostPass &out)
{
    std::vector<Work> work;
    std::vector<int64_t> group_cost;
    {
        size_t total = 0;
        for (int b = 0; b < B; b++) total += (size_t)cdiv(std::max(cu[b + 1] - cu[b], 0), tile_rows);
        work.reserve(total * heads);
        group_cost.reserve((size_t)B * heads);
    }
    std::vector<int64_t> cost;  // of a sequence's tiles, the same for each of its heads
    for (int b = 0; b < B; b++) {
        int32_t s = cu[b + 1] - cu[b];
        if (s <= 0) continue;
        int32_t nt = (int32_t)cdiv(s, tile_rows);
        cost.resize((size_t)nt);
        int64_t gc = 0;
        for (int32_t t = 0; t < nt; t++) {
            if (!key_major) {
                // query tile t: keys 0 .. min(s, (t+1)*tile_rows) - 1 when causal
                int64_t keys = causal ? std::min<int64_t>(s, (int64_t)(t + 1) * tile_rows) : s;
                cost[t] = cdiv(keys, step_rows);
            } else {
                // key tile t: queries from the tile's first key to the end when causal
                int64_t first = causal ? (int64_t)t * tile_rows : 0;
                cost[t] = cdiv(s - first, step_rows) * group_mult;
            }
            gc += cost[t];
        }
        for (int n = 0; n < heads; n++) {
            Work w;
            w.it.seq_start = cu[b];
            w.it.seq_len = s;
            w.it.head = nth_head(n, heads, nq);
            w.group = (int32_t)group_cost.size();
            for (int32_t t = 0; t < nt; t++) {
                w.it.tile = t;
                w.cost = cost[t];
                work.push_back(w);
            }
            group_cost.push_back(gc);
        }
    }
    distribute(work, group_cost, nq, n_wg, tile_rows, out, 0, causal ? 2 * 2 * D : 0, group_mult);  // (two bf16 tensors)
}

// Cuts tiles that would outlast an even share of the pass into parts (see flexsp_item): with W =
// total steps / workgroups, a tile of c steps becomes ceil(c / L) parts of equal length (at most
// kMaxParts, none shorter than kMinPartSteps), where the part length aimed at is L = 3W/4 while that
// is at most kLongPartSteps, then kLongPartSteps, and 0.35 W once that is longer still: a part costs
// its hand-over (a few steps' time) whatever its length, so short parts are kept few and long ones
// are made finer, which evens out the end of the pass.  Longest-first scheduling alone
// finishes no earlier than the longest item, which for a batch of few heads and one dominant
// sequence is several times the even share: the compute units that run out of work wait for it.
// `spare`: tiles of up to this many even shares are left whole (0: every tile longer than a part is cut).
int64_t part_length(int64_t share)
{
    return std::min(share * 3 / 4, std::max<int64_t>(share * 35 / 100, kLongPartSteps));
}
// Parts a tile of c steps is cut into: about `target` steps each, none of fewer than `shortest`.
int part_count(int64_t c, int64_t target, int64_t shortest)
{
    if (c < 2 * shortest || c <= target) return 1;
    return (int)std::min<int64_t>(std::min<int64_t>(cdiv(c, target), kMaxParts), c / shortest);
}
void cut_part(flexsp_item &it, int64_t c, int p, int k, int32_t slot)
{
    it.step_begin = (int32_t)((int64_t)p * c / k);
    it.step_end = (int32_t)((int64_t)(p + 1) * c / k);
    it.slot = slot;
    it.parts = (p << 16) | k;
}
// With a mask, parts of the same number walk about the same rows, parts of one tile do not.  So where a group walks more rows than an
// XCD's L2 holds beside everything else (`row_bytes` of them each, 0 without a mask, kPartAffinityBytes in all), the parts of one number are
// kept on one queue instead of the whole group (`keep`, whose costs are returned).  Not where a pass is little more than a few such groups:
// levelling spreads those over the queues in order of cost, which is the order of their tiles, while parts of one
// number are of few and unequal costs then.  The line lies at three and a half times the largest group, or two and a half where a group is several
// heads, whose parts are about its heads; and none where those are cut into as many parts as there are queues.
// Time of a pass, by group -> by part.  Taken: one sequence of 20 000 tokens, 4 heads, forward 391 -> 373 us, dQ 589 -> 538; 30 721, 12
// heads on 3, dK/dV 5 959 -> 5 227; 12 000, 8 heads on 1, dK/dV 619 -> 570; a mix of 126 120, 1 head, dK/dV 409 -> 370.  Not taken:
// 30 721, 2 heads, forward 426 -> 460, dQ 621 -> 680; 20 000, 3 heads, dQ 405 -> 428; 30 721, 8 heads on 2, dK/dV 3 646 -> 3 832; a mix of
// 68 656 around one of 19 381, 1 head, dQ 195 -> 215; unmasked 6 000, 2 heads on 1, dK/dV 102 -> 116; 12 000, 8 heads, forward 498 -> 530.
// Rows that fit L2: sequences of 3 100 to 5 100 tokens, 2 heads, forward and backward 307 -> 318.  Of 861 passes, drawn and over single
// sequences, which take 1.4 % less by this line, 23 take more than 3 % more; all by part 1.0 % less, 95.
std::vector<int64_t> split_long_items(std::vector<Work> &work, std::vector<int64_t> keep_cost, int n_wg, int spare, int64_t row_bytes, int heads_walked,
                                      HostPass &out)
{
    out.records = 0;
    int64_t total = 0;
    for (Work &w : work) {
        w.keep = w.group;
        w.it.step_begin = 0;
        w.it.step_end = (int32_t)w.cost;
        w.it.slot = -1;
        w.it.parts = 1;
        total += w.cost;
    }
    const int64_t share = total / std::max(n_wg, 1);
    const int64_t target = std::max<int64_t>(part_length(share), kMinPartSteps);
    const size_t n0 = work.size();
    auto parts_of = [&](int64_t c) { return c <= spare * share ? 1 : part_count(c, target, kMinPartSteps); };
    std::vector<int32_t> by_part(keep_cost.size(), -1);  // a cut group's first number beyond the groups'
    int32_t groups_cut = 0;
    int64_t largest = 0, most_parts = 0;
    for (const Work &w : work)
        if (row_bytes * heads_walked * w.it.seq_len > kPartAffinityBytes && parts_of(w.cost) > 1) {
            if (by_part[w.group] < 0) by_part[w.group] = (int32_t)keep_cost.size() + groups_cut++ * kMaxParts;
            largest = std::max(largest, keep_cost[w.group]);
            most_parts = std::max<int64_t>(most_parts, parts_of(w.cost));
        }
    if (2 * total < (heads_walked > 1 ? 5 : 7) * largest && !(heads_walked > 1 && most_parts == kMaxParts)) {
        std::fill(by_part.begin(), by_part.end(), -1);
        groups_cut = 0;
    }
    keep_cost.resize(keep_cost.size() + (size_t)groups_cut * kMaxParts, 0);
    for (size_t i = 0; i < n0; i++) {
        const int64_t c = work[i].cost;
        const int k = parts_of(c);
        if (k < 2 || out.records + k > kMaxSplitRecords) continue;
        const int32_t slot = out.records;
        out.records += k;
        for (int p = 0; p < k; p++) {
            Work w = work[i];
            cut_part(w.it, c, p, k, slot);
            w.cost = w.it.step_end - w.it.step_begin;
            if (by_part[w.group] >= 0) {
                keep_cost[w.group] -= w.cost;
                w.keep = by_part[w.group] + p;
                keep_cost[w.keep] += w.cost;
            }
            if (p == 0)
                work[i] = w;
            else
                work.push_back(w);
        }
    }
    return keep_cost;
}

// Spreads listed work over the queues and orders every queue longest first (see build_pass).
void distribute(std::vector<Work> &work, const std::vector<int64_t> &group_cost, int nq, int n_wg, int tile_rows,
                HostPass &out, int spare, int64_t row_bytes, int heads_walked)
{
    const std::vector<int64_t> keep_cost = split_long_items(work, group_cost, n_wg, spare, row_bytes, heads_walked, out);
    out.steps = out.longest = 0;
    for (const Work &w : work) {
        out.steps += w.cost;
        out.longest = std::max(out.longest, w.cost);
    }
    // what is kept together -> queues
    std::vector<int32_t> order(keep_cost.size());
    for (size_t i = 0; i < order.size(); i++) order[i] = (int32_t)i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t a, int32_t b) { return keep_cost[a] > keep_cost[b]; });
    std::vector<int64_t> load(nq, 0);
    std::vector<int32_t> queue_of(keep_cost.size(), 0);
    for (int32_t g : order) {
        int best = 0;
        for (int x = 1; x < nq; x++)
            if (load[x] < load[best]) best = x;
        queue_of[g] = best;
        load[best] += keep_cost[g];
    }
    // item -> queue: its group's queue.  Each queue's members are kept in order of decreasing
    // cost; the order comes from one stable counting sort of all items (costs are small integers),
    // not from comparison sorts: a plan is built per micro-batch, on the host's time.
    const size_t n = work.size();
    std::vector<int32_t> item_queue(n);
    for (size_t i = 0; i < n; i++) item_queue[i] = queue_of[work[i].keep];
    std::vector<int32_t> by_cost(n);  // item indices, most expensive first, ties in list order
    {
        int64_t maxc = 0;
        for (const Work &w : work) maxc = std::max(maxc, w.cost);
        if (maxc <= (int64_t)(4 * n + 1024)) {
            std::vector<int32_t> start((size_t)maxc + 2, 0);
            for (const Work &w : work) start[(size_t)(maxc - w.cost) + 1]++;
            for (size_t c = 1; c < start.size(); c++) start[c] += start[c - 1];
            for (size_t i = 0; i < n; i++) by_cost[(size_t)start[(size_t)(maxc - work[i].cost)]++] = (int32_t)i;
        } else {  // a few enormous items: the table would be larger than the list
            for (size_t i = 0; i < n; i++) by_cost[i] = (int32_t)i;
            std::stable_sort(by_cost.begin(), by_cost.end(),
                             [&](int32_t a, int32_t b) { return work[a].cost > work[b].cost; });
        }
    }
    std::vector<std::vector<int32_t>> members(nq);
    for (int x = 0; x < nq; x++) members[x].reserve(n / nq + 16);
    for (int32_t idx : by_cost) members[item_queue[idx]].push_back(idx);
    // Level the queues by moving the cheapest items of the fullest queue to the emptiest one (a
    // group that outweighs a whole queue's share, e.g. one dominant sequence with few heads, is
    // split this way; only the moved items lose L2 affinity).
    // Moved items wait in a side list per receiving queue and are merged in once (one insertion
    // into a sorted list per move costs a memmove each, thousands of times when six heavy groups
    // meet eight queues).
    auto dearer = [&](int32_t a, int32_t b) { return work[a].cost > work[b].cost; };
    std::vector<std::vector<int32_t>> incoming(nq);
    auto merge_in = [&](int x) {
        if (incoming[x].empty()) return;
        std::stable_sort(incoming[x].begin(), incoming[x].end(), dearer);
        std::vector<int32_t> merged(members[x].size() + incoming[x].size());
        std::merge(members[x].begin(), members[x].end(), incoming[x].begin(), incoming[x].end(), merged.begin(),
                   dearer);
        members[x].swap(merged);
        incoming[x].clear();
    };
    for (size_t guard = 0; guard < n; guard++) {
        int hi = 0, lo_ = 0;
        for (int x = 1; x < nq; x++) {
            if (load[x] > load[hi]) hi = x;
            if (load[x] < load[lo_]) lo_ = x;
        }
        merge_in(hi);  // (rare: a queue that received items has become the fullest)
        if (members[hi].empty()) break;
        const int32_t cand = members[hi].back();
        const int64_t c = work[cand].cost;
        if (load[hi] - c < load[lo_] + c) break;  // moving would not narrow the gap
        members[hi].pop_back();
        load[hi] -= c;
        load[lo_] += c;
        incoming[lo_].push_back(cand);
    }
    for (int x = 0; x < nq; x++) merge_in(x);
    // Order inside a queue.  Items of long sequences stay longest first.  The tiles of a SHORT sequence
    // (none of more than kGroupMajorSteps steps) are put side by side, where the longest of them would
    // stand: the workgroups of the XCD then take them at about the same time and share the sequence's
    // rows in L2, instead of each meeting them cold (batches of 256- to 1 024-token sequences: 2-4 %
    // faster; no effect where long sequences carry the work).  The queue still ends with its cheapest items.
    {
        std::vector<int64_t> gmax(group_cost.size(), 0);
        for (const Work &w : work) gmax[w.group] = std::max(gmax[w.group], w.cost);
        auto is_short = [&](int32_t g) { return gmax[g] <= kGroupMajorSteps; };
        std::vector<int32_t> count(group_cost.size(), 0), at(group_cost.size(), 0), groups, ordered;
        for (int x = 0; x < nq; x++) {
            // (a queue's members stand dearest first: long sequences' items as they are, in front of the short sequences whose dearest tile costs
            // no more; those by that cost, then one after the other, each one's items as they are.  No sort compares items: plans are
            // made per micro-batch.  With this, a tile's cost taken once for all heads and one list for the forward and the dQ pass, a
            // plan of 82 sequences and 8 heads, 17 408 items, takes 450 us of host time instead of 770, one of 17 and one head 51 instead of 70.)
            std::vector<int32_t> &m = members[x];
            groups.clear();
            for (int32_t i : m)
                if (is_short(work[i].group) && count[work[i].group]++ == 0) groups.push_back(work[i].group);
            std::sort(groups.begin(), groups.end(), [&](int32_t a, int32_t b) { return gmax[a] != gmax[b] ? gmax[a] > gmax[b] : a < b; });
            ordered.resize(m.size());
            int32_t to = 0;
            size_t next = 0;  // the next long sequence's item
            auto longs_from = [&](int64_t cost) {
                for (; next < m.size(); next++) {
                    if (is_short(work[m[next]].group)) continue;
                    if (work[m[next]].cost < cost) break;
                    ordered[to++] = m[next];
                }
            };
            for (int32_t g : groups) {
                longs_from(gmax[g]);
                at[g] = to;
                to += count[g];
                count[g] = 0;
            }
            longs_from(0);
            for (int32_t i : m)
                if (is_short(work[i].group)) ordered[at[work[i].group]++] = i;
            m.swap(ordered);
        }
    }
    out.items.resize(n);
    size_t at = 0;
    for (int x = 0; x <= kMaxQueues; x++) out.offsets[x] = (int64_t)n;
    for (int x = 0; x < nq; x++) {
        out.offsets[x] = (int64_t)at;
        for (int32_t idx : members[x]) out.items[at++] = work[idx].it;
    }
    out.offsets[nq] = (int64_t)n;
    out.tile_rows = tile_rows;
}

// A pass whose items can all be resident at once is launched with one workgroup per item (see ItemDealer).  This lists its
// items in the order of the workgroups: workgroup w runs on XCD w % nq and takes the next item of that queue, or of the
// queue with the most items left where that one has run out.
// Such a pass lasts as long as its longest item, whatever an even share is, so where compute units would be left without
// work its tiles are cut into shorter parts than the plan lists (none when `lowest` is 0): of `lowest` steps or more while
// there is at most one item per compute unit (n_wg counts two), of half of kMinPartSteps or more while all items are resident at
// once and the longest outlasts three shares.  Forward and backward, without -> with: 926 tokens, 8 heads on 4
// 44.5 -> 33.4 us; 440 tokens, 16 heads on 4 62 -> 34 us; 7 616 tokens, 3 heads 159 -> 134 us; 14 938 tokens, 2 heads
// 129 -> 118 us.  (Without the bound on shares 1 480 tokens with 16 heads, which keep the chip busy as they are, took 132
// instead of 124 us.)  The forward's tiles stay as listed: a batch that the plan does not cut gives the same bits as
// flexsp_attn_varlen_fwd_static, and cutting them too is worth 10 % at 7 616 tokens with 3 heads, 0 to 3 % elsewhere.
void direct_list(HostPass &p, int nq, int n_wg, int spare, int64_t lowest)
{
    p.direct.clear();
    if (p.items.empty() || p.items.size() > (size_t)n_wg) return;
    // the tiles, whole, in the order of the queues (a cut one where its first part stands)
    std::vector<int64_t> steps(p.records, 0);
    int64_t total = 0, longest = 0;
    for (const flexsp_item &it : p.items)
        if (it.slot >= 0) steps[it.slot] = std::max<int64_t>(steps[it.slot], it.step_end);
    auto tile_steps = [&](const flexsp_item &it) { return it.slot >= 0 ? steps[it.slot] : (int64_t)it.step_end; };
    auto first_part = [](const flexsp_item &it) { return (it.parts >> 16) == 0; };
    for (const flexsp_item &it : p.items)
        if (first_part(it)) {
            total += tile_steps(it);
            longest = std::max(longest, tile_steps(it));
        }
    const int64_t share = total / n_wg;
    int64_t shortest = 0;
    auto parts_of = [&](int64_t c, int64_t m) { return c <= spare * share ? 1 : part_count(c, std::max(part_length(share), m), m); };
    for (int tier = 0; lowest && !shortest && tier < (longest > 3 * share ? 2 : 1); tier++)
        for (int64_t m = tier == 0 ? lowest : kMinPartSteps / 2; !shortest && m < kMinPartSteps; m += 2) {
            int64_t n = 0;
            for (const flexsp_item &it : p.items)
                if (first_part(it)) n += parts_of(tile_steps(it), m);
            if (n <= (tier == 0 ? n_wg / 2 : n_wg)) shortest = m;
        }
    std::vector<flexsp_item> list;  // the same queues, tiles cut
    list.reserve((size_t)n_wg);
    size_t at[kMaxQueues], end[kMaxQueues];
    int32_t records = 0;
    for (int x = 0; x < nq; x++) {
        at[x] = list.size();
        for (int64_t i = p.offsets[x]; i < p.offsets[x + 1]; i++) {
            flexsp_item it = p.items[i];
            if (!shortest) {
                list.push_back(it);
            } else if (first_part(it)) {
                const int64_t c = tile_steps(it);
                const int k = parts_of(c, shortest);
                for (int part = 0; part < k; part++) {
                    cut_part(it, c, part, k, k > 1 ? records : -1);
                    list.push_back(it);
                }
                if (k > 1) records += k;
            }
        }
        end[x] = list.size();
    }
    if (shortest) p.records = records;
    p.direct.reserve(list.size());
    for (size_t w = 0; w < list.size(); w++) {
        int q = (int)(w % nq);
        if (at[q] == end[q])
            for (int x = 0; x < nq; x++)
                if (end[x] - at[x] > end[q] - at[q]) q = x;
        p.direct.push_back(list[at[q]++]);
    }
}

HalvesCount halves_count(const flexsp_plan *p)
{
    HalvesCount c = {p->T, p->B, 0, 0, 0};
    for (int b = 0; b < p->B; b++) {
        const int64_t n = cdiv(p->cu[b + 1] - p->cu[b], kHalfBq);
        c.tiles += n * p->Hq;
        c.steps += (p->causal ? n * (n + 1) / 2 : n * n) * p->Hq;
        c.longest = std::max(c.longest, n);
    }
    return c;
}

// Whether the forward, launched with one workgroup per item and no tile cut, runs in halves (fwd_halves); if so, its list becomes one of
// halves, a tile's one after the other.
bool halve_items(flexsp_plan *p, int num_cu)
{
    HostPass &f = p->pass[FLEXSP_PASS_FWD];
    const HalvesCount c = halves_count(p);
    if (f.direct.empty() || f.records || !fwd_halves(p->D, c, num_cu)) return false;
    std::vector<flexsp_item> halves;
    halves.reserve((size_t)c.tiles);
    for (flexsp_item it : f.direct)
        for (int i = 0, first = it.tile * (kFwdBq / kHalfBq); i < kFwdBq / kHalfBq && (first + i) * kHalfBq < it.seq_len; i++) {
            it.tile = first + i;
            it.step_end = (int32_t)cdiv(p->causal ? std::min((it.tile + 1) * kHalfBq, it.seq_len) : it.seq_len, kFwdBk);
            halves.push_back(it);
        }
    f.direct.swap(halves);
    return true;
}

// Whether the dK/dV pass takes 128 keys an item (attn_bwd_dkv_wide_kernel; D = 64).  What it gives up: at a walk's start and end, and
// where blocks are masked, its stages run one after the other, a causal walk begins with up to two steps of that kind,
// the last item of a sequence may be half empty, and its items are half as many.  So where walks over the queries are twelve
// steps or more on average, eight if nothing is masked and next to no key empty.  With shorter ones only where its items, one to a workgroup,
// are on the chip at once and those of 64 keys would not be: if query heads have key heads of their own (the walks of several are
// long for so few items), or if nothing is masked and so on.  And not where both passes may run in one launch, which has no such kernel.
// dK/dV pass, 64 keys -> 128.  Taken: sequences of 1 500 tokens, 4 heads, 12 000 tokens not causal 1.34 times as fast, 39 000 1.15, causal 1.13
// and 0.99; 40 000 tokens in sequences of 200, 1 head 1.56; 11 904 in 128, 4 heads 1.71; causal 39 501 in 513, 1 head 1.21.  Not
// taken, in us: 40 000 tokens in 16, 16 heads on 2 97 -> 165; in 129, 8 heads 83 -> 92; in 300, 16 heads on 2 141 -> 168; in 513, 4 heads,
// causal 0.91 times as fast; 12 000 in 1 000, 4 heads on 1, causal 29 -> 47.  544 batches: 5.6 % faster than with 64 keys, nine of them more
// than 3 % slower, the slowest 1.11 times; by the line as it was (five steps for causal walks, none for others) 1.9 % and 197.
bool wide_keys(const flexsp_plan *p, int n_wg)
{
    if (p->D != 64) return false;
    int64_t steps = 0, narrow_steps = 0, walks = 0, items = 0;
    auto walk_steps = [&](int64_t tiles, int64_t all, int64_t skip) { return tiles * all - (p->causal ? tiles * (tiles - 1) / 2 * skip : 0); };
    for (int b = 0; b < p->B; b++) {
        const int64_t s = p->cu[b + 1] - p->cu[b], all = cdiv(s, kDkvBq);
        walks += cdiv(s, kDkvWideBk);
        steps += walk_steps(cdiv(s, kDkvWideBk), all, kDkvWideBk / kDkvBq);
        narrow_steps += walk_steps(cdiv(s, kDkvBk), all, kDkvBk / kDkvBq);
        items += cdiv(s, kDkvBk) * p->Hkv + cdiv(s, kDqBq) * p->Hq;
    }
    if (items <= n_wg) return false;
    const bool full = !p->causal && 40 * steps <= 21 * narrow_steps;
    if (steps >= (full ? 8 : 12) * walks) return true;
    const int64_t wide_items = walks * p->Hkv;
    return 2 * wide_items > n_wg && wide_items <= n_wg && (p->Hq == p->Hkv || full);
}

// Lists the dK/dV and the dQ pass; `forward`: the forward's list, if it is as build_pass has left it.
void list_two_passes(const flexsp_plan *p, const HostPass *forward)
{
    const int nq = p->ctx->num_xcd, n_wg = workgroups_of(p->ctx);
    const bool causal = p->causal != 0;
    static_assert(kFwdBq == kDqBq && kFwdBk == kDqBk, "the forward's and the dQ kernel's items are listed alike");
    HostPass &dkv = p->pass[FLEXSP_PASS_BWD_DKV], &dq = p->pass[FLEXSP_PASS_BWD_DQ];
    build_pass(p->cu, p->B, p->Hkv, p->Hq / p->Hkv, p->wide ? kDkvWideBk : kDkvBk, kDkvBq, causal, true, p->D, nq, n_wg, dkv);
    if (forward)
        dq = *forward;
    else
        build_pass(p->cu, p->B, p->Hq, 1, kDqBq, kDqBk, causal, false, p->D, nq, n_wg, dq);
    direct_list(dkv, nq, n_wg, 0, kShortPartSteps);
    direct_list(dq, nq, n_wg, 0, kShortPartSteps);
}

// The lists of a plan that runs in one pass, when they are asked for (they took most of the time of making it, us: one sequence of 131 072 tokens, 8
// heads 727 -> 251, 49 152 tokens in short ones 337 -> 165, a 64K-token long-tail batch 410 -> 180).
int need_two_passes(const flexsp_plan *p)
{
    if (p->two_listed) return FLEXSP_OK;
    try {
        list_two_passes(p, nullptr);
    } catch (const std::bad_alloc &) {
        p->pass[FLEXSP_PASS_BWD_DKV] = p->pass[FLEXSP_PASS_BWD_DQ] = HostPass{};
        return FLEXSP_OUT_OF_MEMORY;
    }
    p->two_listed = true;
    return FLEXSP_OK;
}

// Whether a backward runs in one pass (attn_bwd_chain.hip): D = 128 and
// - at least two items of 128 keys per compute unit, three steps of 64 query rows an item and head, twelve without a mask: a delta launch in
//   front and the start of an item, during which its compute unit does nothing else, have to be made up for;
// - no item longer than an even share of the steps (0.4 of one where several heads share their keys, whose items are long and few): all
//   compute units wait for the last;
// - no (sequence, kv head) of more than a quarter of the steps: each of its items starts a step or two behind the one before.
// Backward, two kernels -> one pass, us.  Taken: 17 433 tokens, 4 heads, up to 1 290 a sequence 114 -> 88; 28 916 in one, 4 heads 2 776 -> 2 480; 82 128,
// 4 heads, up to 23 445 2 971 -> 2 693; 26 644 in 441, 16 heads on 8 290 -> 279; 66 564 in 757, 8 heads, unmasked (twelve steps an item) 863 -> 823.
// Not taken: 130 077 in one, 1 head 14 965 -> 16 098; 84 931, 1 head, up to 21 776 732 -> 854; 9 400 in 460, 16 heads on 8
// 129 -> 140; 41 048 in 65, 16 heads on 2 321 -> 342; 95 093, 8 heads on 1, unmasked 5 220 -> 6 520; 24 348 in 99, 1 head 19 -> 30.
bool chain_pays(const flexsp_plan *p, int64_t steps, int64_t longest, int64_t largest, int64_t items, int n_cu)
{
    const int64_t G = p->Hq / p->Hkv;
    return items >= 2 * n_cu && steps >= (p->causal ? 3 : 12) * G * items && longest * n_cu * (G > 1 ? 5 : 2) <= 2 * steps && 4 * largest <= steps;
}

struct ChainBundle {
    int32_t cost, team, first, end;
};

// Whether the dies, which take the bundles in this order as they come to an end with one, all have about an even share of the steps: with few
// bundles as dear as each other some take one more than the rest, and everything waits for them.
// Backward, two kernels -> one pass, us, by the largest share over the even one, no mask: 1.00 (32 768 tokens in sequences of 2 048, 8 heads) 881 -> 795; 1.04 (131 072 in
// 1 000, 8 heads) 1 965 -> 1 895; 1.08 (49 352 in one, 16 heads on 4) 60 230 -> 60 950; 1.2 (65 536 in 1 600, 4 heads) 721 -> 728, (20 000 in 1 500, 8 heads)
// 413 -> 495; 1.3 (40 000 in 3 000, 12 heads on 4) 2 270 -> 2 680.  With a mask later bundles are cheaper, and the pass gains more: forward, backward and permutes
// at 1.08 (121 707, up to 1 606 a sequence, 2 heads) 469 -> 451, at 1.12 (124 314 in 433, 4 heads on 2) 739 -> 739.
bool dies_even(const std::vector<flexsp_item> &list, const std::vector<ChainBundle> &bundles, int dies, bool causal)
{
    std::vector<int64_t> share((size_t)dies, 0);
    int64_t all = 0;
    for (const ChainBundle &b : bundles) {
        int64_t steps = 0;
        for (int32_t i = b.first; i < b.end; i++) steps += list[i].step_end;
        *std::min_element(share.begin(), share.end()) += steps;
        all += steps;
    }
    return 100 * *std::max_element(share.begin(), share.end()) * dies <= (causal ? 111 : 106) * all;
}

// Lists a backward in one pass, if it is one.  The list's bundles (see chain_take) are what a compute die's workgroups, one per compute
// unit, work on at a time, and what they share should stay in its L2: the rows of dQ that are added to, Q and dO, 64 KB a step.  So a long
// sequence's key tiles are bundles of up to kChainTeam, one to a workgroup, which go through the steps one behind the other; heads and
// sequences of fewer tiles are put together, kChainSpan items or a little more, and lie in a bundle as their walks' lengths say, so that
// an item does not stand right behind the one that it follows.  Bundles, too, stand dearest first.  Items of a (sequence, kv head) then stand in the
// order of their keys, which is what they wait for.
// Backward by kChainSpan, us, 1 / 32 / 64 / 128 / 256 / no bound: sequences of 4 096 tokens, 8 heads 1 744 / 1 744 / 1 700 / 1 695 / 1 797 / 2 006;
// 1 024 514 / 476 / 462 / 459 / 490 / 521; a 64K-token long-tail batch 1 263 / 1 247 / 1 244 / 1 266 / 1 274 / 1 274.
// An item's fields here: step_begin the bundle's first key tile of this (sequence, kv head), step_end its steps, slot the first of its
// sequence's query tiles among all that several key tiles add to, parts whether the next key tile is in another bundle.
void build_chain(flexsp_plan *p, int n_cu)
{
    if (p->D != 128) return;
    const int G = p->Hq / p->Hkv, skip = p->causal ? kChainBk / kDkvBq : 0;  // steps a walk is shorter than that of the key tile in front
    struct Seq {
        int64_t cost;
        int32_t b, base;
    };
    std::vector<Seq> seqs;
    int64_t tiles = 0, steps = 0, longest = 0, largest = 0, items = 0;
    for (int b = 0; b < p->B; b++) {
        const int64_t s = p->cu[b + 1] - p->cu[b], nt = cdiv(s, kDkvBq), nb = cdiv(s, kChainBk);
        if (s <= 0) continue;
        const int64_t cost = (nb * nt - nb * (nb - 1) / 2 * skip) * G;
        seqs.push_back(Seq{cost, b, (int32_t)tiles});
        if (nb > 1) tiles += nt;  // (rows that one key tile sees alone are not kept)
        steps += cost * p->Hkv;
        items += nb * p->Hkv;
        longest = std::max(longest, nt * G);
        largest = std::max(largest, cost);
    }
    if (!chain_pays(p, steps, longest, largest, items, n_cu) || tiles * p->Hq > kChainMostTiles) return;
    std::stable_sort(seqs.begin(), seqs.end(), [](const Seq &a, const Seq &b) { return a.cost > b.cost; });
    std::vector<ChainBundle> bundles;
    std::vector<flexsp_item> list;
    list.reserve((size_t)items);
    int32_t open = 0;  // first item of the bundle that is being filled
    auto close = [&](int32_t team) {
        if ((size_t)open == list.size()) return;
        std::stable_sort(list.begin() + open, list.end(), [](const flexsp_item &a, const flexsp_item &b) { return a.step_end > b.step_end; });
        bundles.push_back(ChainBundle{list[open].step_end, team, open, (int32_t)list.size()});
        open = (int32_t)list.size();
    };
    for (const Seq &q : seqs)
        for (int32_t g = 0; g < p->Hkv; g++) {
            const int32_t s = p->cu[q.b + 1] - p->cu[q.b], nt = (int32_t)cdiv(s, kDkvBq), nb = (int32_t)cdiv(s, kChainBk);
            const int32_t teams = (int32_t)cdiv(nb, kChainTeam);
            if (teams > 1) close(0);
            for (int32_t t = 0; t < teams; t++) {
                const int32_t from = (int32_t)((int64_t)t * nb / teams), to = (int32_t)((int64_t)(t + 1) * nb / teams);
                for (int32_t i = from; i < to; i++)
                    list.push_back(flexsp_item{p->cu[q.b], s, i, g, from, (nt - i * skip) * G, q.base, i + 1 == to && to < nb});
                if (teams > 1) close(t);
            }
            if ((int64_t)list.size() - open >= kChainSpan) close(0);
        }
    close(0);
    std::stable_sort(bundles.begin(), bundles.end(), [](const ChainBundle &a, const ChainBundle &b) { return a.cost != b.cost ? a.cost > b.cost : a.team < b.team; });
    if (!dies_even(list, bundles, std::max(1, n_cu / kChainTeam), p->causal)) return;
    p->chain.reserve(list.size());
    p->chain_bundles.reserve(bundles.size() + 1);
    for (const ChainBundle &b : bundles) {
        p->chain_bundles.push_back((int32_t)p->chain.size());
        p->chain.insert(p->chain.end(), list.begin() + b.first, list.begin() + b.end);
    }
    p->chain_bundles.push_back((int32_t)p->chain.size());
    p->chain_tiles = tiles * p->Hq;
}

int check_attn_common(flexsp_ctx *ctx, flexsp_plan *plan, const int32_t *cu_dev, int32_t head_begin,
                      int32_t head_count, int32_t kv_head_begin, int32_t kv_head_count, int causal)
{
    (void)cu_dev;  // the plan carries the lengths; the device copy is not read by the plan-based calls
    if (!ctx || !plan) return FLEXSP_INVALID_ARGUMENT;
    if (plan->ctx != ctx || plan->kvshard) return FLEXSP_PLAN_MISMATCH;
    if (head_begin < 0 || kv_head_begin < 0 || head_count <= 0 || kv_head_count <= 0)
        return FLEXSP_INVALID_ARGUMENT;
    if (head_count % kv_head_count != 0) return FLEXSP_INVALID_ARGUMENT;
    if (head_count != plan->Hq || kv_head_count != plan->Hkv || (causal != 0) != (plan->causal != 0))
        return FLEXSP_PLAN_MISMATCH;
    if (ctx->device < 0 || !plan->dev_base) return FLEXSP_NO_DEVICE;
    return FLEXSP_OK;
}

// Puts a freshly built plan's queues on the device (nothing to do for a host-only context): one
// slab, carved into [items x3][offsets x3][counters x3][delta, lse2], and what a backward in one pass needs instead of the two
// passes'.  Items of a key-shard plan are written in their wider device form.  On failure the plan is deleted and a status returned.
int plan_upload(flexsp_ctx *ctx, flexsp_plan *p)
{
    for (int i = 0; i < 3; i++) std::memset(&p->dq[i], 0, sizeof(PassQueues));
    if (ctx->device < 0) return FLEXSP_OK;
    const size_t item_bytes = p->kvshard ? sizeof(flexsp_shard_item) : sizeof(flexsp_item);
    {

        // one allocation: [items x3][offsets x3][counters x3][delta]
        int nq = ctx->num_xcd;
        auto on_device = [&](int i) { return i == FLEXSP_PASS_FWD || p->chain.empty(); };
        size_t off = 0, item_off[3], offs_off[3], ctr_off[3];
        auto align = [](size_t x) { return (x + 255) & ~(size_t)255; };
        for (int i = 0; i < 3; i++) {
            item_off[i] = off;
            if (on_device(i)) off = align(off + std::max(p->pass[i].items.size(), p->pass[i].direct.size()) * item_bytes);
        }
        for (int i = 0; i < 3; i++) {
            offs_off[i] = off;
            off = align(off + (nq + 1) * sizeof(int32_t));
        }
        for (int i = 0; i < 3; i++) {
            ctr_off[i] = off;
            off = align(off + (nq + 1) * kCounterStride * sizeof(int32_t));
        }
        size_t flag_off[3], part_off[3];
        for (int i = 0; i < 3; i++) {
            flag_off[i] = off;
            if (on_device(i)) off = align(off + (size_t)p->pass[i].records * sizeof(int32_t));
        }
        // (a chain's dealer and flags are cleared by the launch in front of it)
        const size_t chain_tiles = p->chain.empty() ? 0 : (size_t)p->chain_tiles;
        const size_t chain_items_off = off;
        off = align(off + p->chain.size() * sizeof(flexsp_item));
        const size_t chain_offs_off = off;
        off = align(off + (p->chain.empty() ? 0 : p->chain_bundles.size()) * sizeof(int32_t));
        size_t head_bytes = off;
        const size_t chain_ctr_off = off, chain_flag_off = off + (1 + kChainDies) * kCounterStride * sizeof(int32_t);
        if (!p->chain.empty()) off = align(chain_flag_off + chain_tiles * sizeof(int32_t));
        const size_t chain_rows_off = off;
        off = align(off + chain_tiles * kChainTileBytes);
        size_t delta_off = off;
        off = align(off + p->delta_bytes + 512);  // the dK/dV kernel reads up to 63 floats past a row's end
        for (int i = 0; i < 3; i++) {
            part_off[i] = off;
            if (on_device(i)) off = align(off + (size_t)p->pass[i].records * kPartialBytes);
        }
        hipError_t e = hipSetDevice(ctx->device);
        if (e == hipSuccess) e = slab_get(ctx, off ? off : 256, head_bytes ? head_bytes : 256, p->slab);
        if (e == hipErrorOutOfMemory && !p->chain.empty()) {  // two passes need less
            (void)hipGetLastError();
            p->chain.clear();
            if (const int rc = need_two_passes(p)) {
                delete p;
                return rc;
            }
            return plan_upload(ctx, p);
        }
        if (e != hipSuccess) {
            delete p;
            return hip_fail(e);
        }
        p->dev_base = p->slab.dev;
        p->dev_bytes = off;
        char *stage = (char *)p->slab.host;
        std::memset(stage, 0, head_bytes);  // also the ticket counters: every plan starts with them clear
        for (int i = 0; i < 3; i++) {
            if (!on_device(i)) continue;
            const bool direct = !p->pass[i].direct.empty();
            const std::vector<flexsp_item> &items = direct ? p->pass[i].direct : p->pass[i].items;
            if (p->kvshard) {
                // the host list names a sequence by its index (seq_start); the device item carries its ranges
                flexsp_shard_item *d = (flexsp_shard_item *)(stage + item_off[i]);
                for (size_t n = 0; n < items.size(); n++) {
                    const flexsp_item &it = items[n];
                    const int b = it.seq_start;
                    // a part of a cut tile: the keys of its steps only, positions counted from its first key
                    // (the dK/dV pass finds a part's steps itself)
                    const int32_t np = it.parts & 0xffff, part = it.parts >> 16;
                    const bool by_keys = np > 1 && i != FLEXSP_PASS_BWD_DKV;
                    const int32_t skip = by_keys ? it.step_begin * kFwdBk : 0;
                    int32_t k_len = p->cu_k[b + 1] - p->cu_k[b];
                    if (by_keys && part + 1 < np) k_len = std::min(k_len, it.step_end * kFwdBk);
                    d[n] = flexsp_shard_item{p->cu[b], p->cu[b + 1] - p->cu[b], p->cu_k[b] + skip, k_len - skip,
                                             p->shift[b] - skip, it.tile, it.head | (part << 16) | (np << 24), it.slot};
                }
            } else if (!items.empty()) {
                std::memcpy(stage + item_off[i], items.data(), items.size() * sizeof(flexsp_item));
            }
            int32_t *o = (int32_t *)(stage + offs_off[i]);
            for (int x = 0; x <= nq; x++) o[x] = (int32_t)p->pass[i].offsets[x];
            p->dq[i].items = (const flexsp_item *)((char *)p->dev_base + item_off[i]);
            p->dq[i].offsets = (const int32_t *)((char *)p->dev_base + offs_off[i]);
            p->dq[i].counters = (int32_t *)((char *)p->dev_base + ctr_off[i]);
            p->dq[i].nq = nq;
            p->dq[i].direct = direct ? 1 : 0;
            p->dq[i].split_flags = (int32_t *)((char *)p->dev_base + flag_off[i]);
            p->dq[i].split_scratch = (char *)p->dev_base + part_off[i];
        }
        if (!p->chain.empty()) {
            std::memcpy(stage + chain_items_off, p->chain.data(), p->chain.size() * sizeof(flexsp_item));
            std::memcpy(stage + chain_offs_off, p->chain_bundles.data(), p->chain_bundles.size() * sizeof(int32_t));
            std::memset(&p->chain_dq, 0, sizeof(PassQueues));
            p->chain_dq.items = (const flexsp_item *)((char *)p->dev_base + chain_items_off);
            p->chain_dq.offsets = (const int32_t *)((char *)p->dev_base + chain_offs_off);
            p->chain_dq.counters = (int32_t *)((char *)p->dev_base + chain_ctr_off);
            p->chain_dq.nq = (int32_t)p->chain_bundles.size() - 1;
            p->chain_dq.split_flags = (int32_t *)((char *)p->dev_base + chain_flag_off);
            p->chain_dq.split_scratch = (char *)p->dev_base + chain_rows_off;
        }
        // asynchronous upload on the context's own stream, after the kernels of the slab's previous
        // plan; the hot calls make their stream wait for `ready` (or find it complete already)
        if (p->slab.done_valid) e = hipStreamWaitEvent(ctx->upload, p->slab.done, 0);
        if (e == hipSuccess && head_bytes)
            e = hipMemcpyAsync(p->dev_base, stage, head_bytes, hipMemcpyHostToDevice, ctx->upload);
        if (e == hipSuccess) e = hipEventRecord(p->slab.ready, ctx->upload);
        if (e != hipSuccess) {
            (void)hipStreamSynchronize(ctx->upload);
            ctx->slab_bytes -= p->slab.dev_bytes;
            slab_free(p->slab);
            ctx->slabs_owned--;
            delete p;
            return hip_fail(e);
        }
        p->slab.done_valid = false;
        p->delta = (float *)((char *)p->dev_base + delta_off);
    }
    return FLEXSP_OK;
}

// Whether no output of a backward shares memory with one of its inputs (the views' extents: interleaved views count as
// sharing).
bool outputs_apart(const flexsp_plan *p, const AttnArgs &a)
{
    struct Bytes {
        uintptr_t lo, hi;
    };
    auto view = [&](const void *first, int64_t T, int64_t st, int64_t heads, int64_t sh, int64_t eb) {
        const uintptr_t lo = (uintptr_t)first;
        return Bytes{lo, T > 0 ? lo + (uintptr_t)(((T - 1) * st + (heads - 1) * sh + p->D) * eb) : lo};
    };
    const int64_t Tk = p->kvshard ? p->Tk : p->T, gb = a.grad_f32 ? 4 : 2;
    const Bytes in[] = {view(a.q, p->T, a.q_st, p->Hq, a.q_sh, 2),    view(a.k, Tk, a.k_st, p->Hkv, a.k_sh, 2),
                        view(a.v, Tk, a.v_st, p->Hkv, a.v_sh, 2),     view(a.o, p->T, a.o_st, p->Hq, a.o_sh, 2),
                        view(a.dO, p->T, a.do_st, p->Hq, a.do_sh, 2), {(uintptr_t)a.lse_in, (uintptr_t)(a.lse_in + p->T * p->Hq)}};
    const Bytes out[] = {view(a.dq, p->T, a.dq_st, p->Hq, a.dq_sh, gb), view(a.dk, Tk, a.dk_st, p->Hkv, a.dk_sh, gb),
                         view(a.dv, Tk, a.dv_st, p->Hkv, a.dv_sh, gb)};
    for (const Bytes &x : in)
        for (const Bytes &y : out)
            if (x.lo < y.hi && y.lo < x.hi) return false;
    return true;
}

// Backwards that run their two passes in one launch (see attn_bwd_both_kernel): those whose items can all be resident at
// once, and whose outputs lie apart from their inputs: side by side, one pass would read what the other has already
// overwritten, where one after the other dq over o and dk, dv over k, v come out right.  (Up to twice as many: 3 500 tokens with 3 heads 156 -> 152 us, but 1 480 tokens with 16 heads 125 -> 132 us.)
// Fills in what such a launch needs and returns its grid (each pass's workgroups keep to their XCD: the dQ pass starts at a
// multiple of the number of queues), or 0.
int both_at_once(const flexsp_ctx *ctx, const flexsp_plan *p, AttnArgs &a)
{
    const int dkv = (int)p->pass[FLEXSP_PASS_BWD_DKV].direct.size(), dq = (int)p->pass[FLEXSP_PASS_BWD_DQ].direct.size();
    // (a plan of 128 keys an item may fit here, because its items are half as many, but the single launch has no such kernel)
    if (p->wide || !dkv || !dq || dkv + dq > workgroups_of(ctx) || !outputs_apart(p, a)) return 0;
    a.pq = p->dq[FLEXSP_PASS_BWD_DKV];
    a.dq_pq = p->dq[FLEXSP_PASS_BWD_DQ];
    a.dkv_items = dkv;
    a.dq_wg = (int)cdiv(dkv, ctx->num_xcd) * ctx->num_xcd;
    const int grid = a.dq_wg + dq;
    a.delta_out = a.lse_out = nullptr;  // (the dK/dV pass forms its own)
    return grid;
}

int grid_for(const flexsp_ctx *ctx, const HostPass &p, int per_cu)
{
    if (!p.direct.empty()) return (int)p.direct.size();
    return p.items.empty() ? 1 : ctx->num_cu * per_cu;
}

// Workgroups per compute unit of a backward pass.  With D = 64 three fit (dQ 164 registers, dK/dV of 64 keys 147, 42 KB of LDS) and
// hide more of each other's waits, but each is slower: where the longest item is most of a workgroup's share, the others wait for it.
// dQ, two -> three: 30 011 tokens, 12 heads on 4, not causal 316 -> 299 us (longest item 0.3 of a share); causal sequences of 4 096 tokens,
// 8 heads 418 -> 378 (a quarter); 21 751 tokens, 4 heads 66.6 -> 68.8 (a whole share).  dK/dV: 65 536 tokens in causal sequences of 512,
// 8 heads 152 -> 127; 31 860 tokens in sequences of 300 to 600, 8 heads on 4 72 -> 66 (half a share).  D = 128 and dK/dV of 128 keys need the
// registers of two.
int bwd_per_cu(const flexsp_ctx *ctx, const flexsp_plan *plan, int pass)
{
    const HostPass &p = plan->pass[pass];
    if (plan->wide && pass == FLEXSP_PASS_BWD_DKV) return 2;  // (its registers)
    return plan->D == 64 && 2 * p.longest * workgroups_of(ctx) <= p.steps ? 3 : 2;
}

// ... and of a forward, likewise: with D = 64 three (163 registers, 33 KB of LDS).  65 536 tokens, 8 heads, two -> three: causal sequences of
// 256 tokens 64 -> 58 us, 1 024 117 -> 105, 4 096 304 -> 289; not causal 256 78 -> 69, 1 024 168 -> 153, 2 048 284 -> 273, 16 384 2 129 -> 2 018
// (with the backward behind it 8 741 -> 8 658); 30 011 tokens, 12 heads on 4, not causal 237 -> 225.
int fwd_per_cu(const flexsp_ctx *ctx, const flexsp_plan *plan)
{
    const HostPass &p = plan->pass[FLEXSP_PASS_FWD];
    const bool even = 2 * p.longest * workgroups_of(ctx) <= p.steps;
    return plan->D == 64 && even ? 3 : 2;
}

}  // namespace

namespace flexsp {
int ctx_device(const flexsp_ctx *ctx) { return ctx ? ctx->device : -1; }
int hip_status(hipError_t e) { return hip_fail(e); }
}  // namespace flexsp

extern "C" {

const char *flexsp_strerror(int status)
{
    switch (status) {
    case FLEXSP_OK: return "ok";
    case FLEXSP_INVALID_ARGUMENT: return "invalid argument";
    case FLEXSP_UNSUPPORTED: return "unsupported configuration";
    case FLEXSP_PLAN_MISMATCH: return "arguments do not match the plan";
    case FLEXSP_HIP_ERROR: return "HIP runtime error";
    case FLEXSP_OUT_OF_MEMORY: return "out of memory";
    case FLEXSP_NO_DEVICE: return "no usable gfx950 device";
    default: return "unknown status";
    }
}

int flexsp_last_hip_error(void) { return g_last_hip_error; }

const char *flexsp_version(void) { return "0.1"; }

int flexsp_ctx_create(flexsp_ctx **out, int device)
{
    if (!out || device < -1) return FLEXSP_INVALID_ARGUMENT;
    *out = nullptr;
    flexsp_ctx *c = new (std::nothrow) flexsp_ctx;
    if (!c) return FLEXSP_OUT_OF_MEMORY;
    c->device = device;
    c->num_cu = 0;
    c->num_xcd = kMaxQueues;
    c->profiling = false;
    c->events_used = 0;
    c->dropped = 0;
    if (device >= 0) {
        int n = 0;
        hipError_t e = hipGetDeviceCount(&n);
        if (e != hipSuccess || device >= n) {
            delete c;
            g_last_hip_error = (int)e;
            return FLEXSP_NO_DEVICE;
        }
        hipDeviceProp_t pr;
        e = hipGetDeviceProperties(&pr, device);
        if (e != hipSuccess) {
            delete c;
            return hip_fail(e);
        }
        if (std::strncmp(pr.gcnArchName, "gfx950", 6) != 0) {
            delete c;
            return FLEXSP_NO_DEVICE;
        }
        c->num_cu = pr.multiProcessorCount;
        e = hipSetDevice(device);
        if (e == hipSuccess) e = hipStreamCreateWithFlags(&c->upload, hipStreamNonBlocking);
        if (e == hipSuccess) e = static_scratch_init(device);  // this device is current here
        if (e != hipSuccess) {
            if (c->upload) (void)hipStreamDestroy(c->upload);
            delete c;
            return hip_fail(e);
        }
    }
    *out = c;
    return FLEXSP_OK;
}

void flexsp_ctx_destroy(flexsp_ctx *ctx)
{
    if (!ctx) return;
    if (ctx->device >= 0) (void)hipSetDevice(ctx->device);
    for (EventPair &e : ctx->events) {
        (void)hipEventDestroy(e.start);
        (void)hipEventDestroy(e.stop);
    }
    if (ctx->device >= 0) {
        if (!ctx->slabs.empty()) (void)hipDeviceSynchronize();  // kernels of destroyed plans may still run
        for (PlanSlab &s : ctx->slabs) slab_free(s);
        if (ctx->upload) (void)hipStreamDestroy(ctx->upload);
    }
    delete ctx;
}

int flexsp_profile_start(flexsp_ctx *ctx, int32_t max_launches)
{
    if (!ctx || max_launches <= 0) return FLEXSP_INVALID_ARGUMENT;
    if (ctx->device < 0) return FLEXSP_NO_DEVICE;
    try {
        ctx->events.reserve((size_t)max_launches);
    } catch (const std::bad_alloc &) {
        return FLEXSP_OUT_OF_MEMORY;
    }
    {
        hipError_t r = hipSetDevice(ctx->device);  // events belong to the device that is current when they are made
        if (r != hipSuccess) return hip_fail(r);
    }
    while (ctx->events.size() < (size_t)max_launches) {
        EventPair e;
        e.kernel = 0;
        hipError_t r = hipEventCreate(&e.start);
        if (r != hipSuccess) return hip_fail(r);
        r = hipEventCreate(&e.stop);
        if (r != hipSuccess) {
            (void)hipEventDestroy(e.start);
            return hip_fail(r);
        }
        ctx->events.push_back(e);
    }
    ctx->events_used = 0;
    ctx->dropped = 0;
    ctx->profiling = true;
    return FLEXSP_OK;
}

int flexsp_profile_stop(flexsp_ctx *ctx, flexsp_profile *out)
{
    if (!ctx || !out) return FLEXSP_INVALID_ARGUMENT;
    if (ctx->device < 0) return FLEXSP_NO_DEVICE;
    std::memset(out, 0, sizeof(*out));
    ctx->profiling = false;
    for (size_t i = 0; i < ctx->events_used; i++) {
        EventPair &e = ctx->events[i];
        hipError_t r = hipEventSynchronize(e.stop);
        if (r != hipSuccess) return hip_fail(r);
        float ms = 0.f;
        r = hipEventElapsedTime(&ms, e.start, e.stop);
        if (r != hipSuccess) return hip_fail(r);
        out->ms[e.kernel] += ms;
        out->launches[e.kernel]++;
    }
    out->dropped = ctx->dropped;
    ctx->events_used = 0;
    return FLEXSP_OK;
}

int flexsp_ctx_num_cu(const flexsp_ctx *ctx) { return ctx ? ctx->num_cu : 0; }
int flexsp_ctx_num_xcd(const flexsp_ctx *ctx) { return ctx ? ctx->num_xcd : 0; }

int flexsp_plan_create(flexsp_ctx *ctx, const int32_t *cu, int32_t B, int32_t Hq, int32_t Hkv,
                       int32_t D, int causal, flexsp_plan **out)
{
    if (!out) return FLEXSP_INVALID_ARGUMENT;
    *out = nullptr;
    if (!ctx || !cu || B < 0 || Hq <= 0 || Hkv <= 0 || D <= 0) return FLEXSP_INVALID_ARGUMENT;
    if (Hq % Hkv != 0) return FLEXSP_INVALID_ARGUMENT;
    if (cu[0] != 0) return FLEXSP_INVALID_ARGUMENT;
    for (int b = 0; b < B; b++)
        if (cu[b + 1] < cu[b]) return FLEXSP_INVALID_ARGUMENT;
    if (D != 64 && D != 128) return FLEXSP_UNSUPPORTED;
    flexsp_plan *p = new (std::nothrow) flexsp_plan;
    if (!p) return FLEXSP_OUT_OF_MEMORY;
    p->ctx = ctx;
    p->B = B; p->Hq = Hq; p->Hkv = Hkv; p->D = D; p->causal = causal ? 1 : 0;
    p->T = cu[B];
    p->dev_base = nullptr; p->dev_bytes = 0; p->delta = nullptr;
    p->uploaded = false; p->used = false; p->multi_stream = false; p->last_stream = nullptr;
    p->delta_bytes = 2 * (size_t)p->T * Hq * sizeof(float);  // delta and log2-domain LSE, [Hq, T] each
    try {
        p->cu.assign(cu, cu + B + 1);
        const int nq = ctx->num_xcd, n_wg = workgroups_of(ctx);
        build_pass(p->cu, B, Hq, 1, kFwdBq, kFwdBk, causal != 0, false, D, nq, n_wg, p->pass[FLEXSP_PASS_FWD]);
        p->wide = wide_keys(p, n_wg);
        build_chain(p, n_wg / 2);
        p->two_listed = p->chain.empty();
        if (p->two_listed) list_two_passes(p, &p->pass[FLEXSP_PASS_FWD]);
        direct_list(p->pass[FLEXSP_PASS_FWD], nq, n_wg, 0, 0);
        p->halves = halve_items(p, n_wg / 2);
    } catch (const std::bad_alloc &) {
        delete p;
        return FLEXSP_OUT_OF_MEMORY;
    }
    {
        int rc = plan_upload(ctx, p);
        if (rc) return rc;
    }
    *out = p;
    return FLEXSP_OK;
}

int flexsp_plan_create_kvshard(flexsp_ctx *ctx, const int32_t *cu_q, const int32_t *cu_k, const int32_t *shift,
                               int32_t B, int32_t Hq, int32_t Hkv, int32_t D, int causal, flexsp_plan **out)
{
    if (!out) return FLEXSP_INVALID_ARGUMENT;
    *out = nullptr;
    if (!ctx || !cu_q || !cu_k || (!shift && B > 0) || B < 0 || Hq <= 0 || Hkv <= 0 || D <= 0)
        return FLEXSP_INVALID_ARGUMENT;
    if (Hq % Hkv != 0 || cu_q[0] != 0 || cu_k[0] != 0) return FLEXSP_INVALID_ARGUMENT;
    for (int b = 0; b < B; b++) {
        if (cu_q[b + 1] < cu_q[b] || cu_k[b + 1] < cu_k[b]) return FLEXSP_INVALID_ARGUMENT;
        // positions are token counts: |shift| beyond 2^30 would overflow the kernels' 32-bit arithmetic
        if (shift[b] > (1 << 30) || shift[b] < -(1 << 30)) return FLEXSP_INVALID_ARGUMENT;
    }
    if (D != 64 && D != 128) return FLEXSP_UNSUPPORTED;
    if (Hq > 0xffff) return FLEXSP_UNSUPPORTED;  // a device item keeps the head in 16 bits
    flexsp_plan *p = new (std::nothrow) flexsp_plan;
    if (!p) return FLEXSP_OUT_OF_MEMORY;
    p->ctx = ctx;
    p->B = B; p->Hq = Hq; p->Hkv = Hkv; p->D = D; p->causal = causal ? 1 : 0;
    p->T = cu_q[B];
    p->Tk = cu_k[B];
    p->kvshard = true;
    p->dev_base = nullptr; p->dev_bytes = 0; p->delta = nullptr;
    p->uploaded = false; p->used = false; p->multi_stream = false; p->last_stream = nullptr;
    p->delta_bytes = 2 * (size_t)p->T * Hq * sizeof(float);  // delta and log2-domain LSE of the query rows
    static_assert(kFwdBq == kDqBq && kFwdBk == kDqBk, "the forward's and the dQ kernel's shard items are listed alike");
    try {
        p->cu.assign(cu_q, cu_q + B + 1);
        p->cu_k.assign(cu_k, cu_k + B + 1);
        p->shift.assign(shift, shift + B);
        // forward and dQ kernel: items (sequence index, query tile, head); cost = key tiles the tile's rows can see
        {
            std::vector<Work> work;
            std::vector<int64_t> group_cost;
            for (int b = 0; b < B; b++) {
                const int32_t sq = cu_q[b + 1] - cu_q[b], sk = cu_k[b + 1] - cu_k[b];
                if (sq <= 0) continue;
                const int32_t nt = (int32_t)cdiv(sq, kFwdBq);
                for (int n = 0; n < Hq; n++) {
                    const int h = nth_head(n, Hq, ctx->num_xcd);
                    const int32_t gid = (int32_t)group_cost.size();
                    int64_t gc = 0;
                    for (int32_t t = 0; t < nt; t++) {
                        int64_t keys = sk;
                        if (causal) keys = std::max<int64_t>(0, std::min<int64_t>(sk, (int64_t)(t + 1) * kFwdBq + shift[b]));
                        Work w;
                        w.it.seq_start = b;  // the sequence INDEX (see plan_upload); its ranges are in cu / cu_k / shift
                        w.it.seq_len = sq;
                        w.it.tile = t;
                        w.it.head = h;
                        w.cost = cdiv(keys, kFwdBk) + 1;  // an item without visible keys still writes its rows
                        w.group = gid;
                        work.push_back(w);
                        gc += w.cost;
                    }
                    group_cost.push_back(gc);
                }
            }
            // (a tile is cut only when it would outlast TWO even shares: with a share of a few dozen steps, as
            // on a micro-batch split over a ring, the hand-over of the parts costs more than the wait for a
            // tile that is a little longer than the rest)
            distribute(work, group_cost, ctx->num_xcd, workgroups_of(ctx), kFwdBq, p->pass[FLEXSP_PASS_FWD], 2);
            p->pass[FLEXSP_PASS_BWD_DQ] = p->pass[FLEXSP_PASS_FWD];
        }
        // dK/dV kernel: items (sequence index, key tile of the shard, kv head); cost = steps of 64 query rows
        // from the first row that sees the tile, for every query head of the group.
        {
            std::vector<Work> work;
            std::vector<int64_t> group_cost;
            const int G = Hq / Hkv;
            for (int b = 0; b < B; b++) {
                const int32_t sq = cu_q[b + 1] - cu_q[b], sk = cu_k[b + 1] - cu_k[b];
                if (sk <= 0) continue;
                const int32_t nt = (int32_t)cdiv(sk, kDkvBk);
                for (int g = 0; g < Hkv; g++) {
                    const int32_t gid = (int32_t)group_cost.size();
                    int64_t gc = 0;
                    for (int32_t t = 0; t < nt; t++) {
                        int64_t qfirst = 0;
                        if (causal) qfirst = std::max<int64_t>(0, (int64_t)t * kDkvBk - shift[b]) / kDkvBq * kDkvBq;
                        Work w;
                        w.it.seq_start = b;
                        w.it.seq_len = sk;
                        w.it.tile = t;
                        w.it.head = g;
                        w.cost = std::max<int64_t>(0, cdiv((int64_t)sq - qfirst, kDkvBq)) * G + 1;  // (the rows are written even if nobody sees them)
                        w.group = gid;
                        work.push_back(w);
                        gc += w.cost;
                    }
                    group_cost.push_back(gc);
                }
            }
            // Cut like the query tiles.  (They were not: few key heads with several query heads each, or one long sequence,
            // are fewer tiles than workgroups, and a tile is a chain of all its group's heads.  One device's ring pass, whole tiles ->
            // cut: 14 514 tokens over four devices, 16 heads on 2 1 222 -> 622 us; 2 517, 8 heads on 1 199 -> 132; 4 912 over two, 2
            // heads, D = 64 158 -> 102; 35 804 over eight, 16 heads on 4 4 949 -> 4 563; 5 306 over four, 2 heads 180 -> 162.)
            distribute(work, group_cost, ctx->num_xcd, workgroups_of(ctx), kDkvBk, p->pass[FLEXSP_PASS_BWD_DKV], 2);
        }
        for (int i = 0; i < 3; i++)
            direct_list(p->pass[i], ctx->num_xcd, workgroups_of(ctx), 2, i == FLEXSP_PASS_FWD ? 0 : kShortPartSteps);
    } catch (const std::bad_alloc &) {
        delete p;
        return FLEXSP_OUT_OF_MEMORY;
    }
    {
        int rc = plan_upload(ctx, p);
        if (rc) return rc;
    }
    *out = p;
    return FLEXSP_OK;
}

void flexsp_plan_destroy(flexsp_plan *plan)
{
    if (!plan) return;
    if (plan->dev_base) {
        flexsp_ctx *ctx = plan->ctx;
        (void)hipSetDevice(ctx->device);
        PlanSlab s = plan->slab;
        // whoever gets this slab next must come after the kernels still running on it
        s.done_valid = false;
        if (plan->used) {
            if (plan->multi_stream || hipEventRecord(s.done, plan->last_stream) != hipSuccess)
                (void)hipDeviceSynchronize();
            else
                s.done_valid = true;
        }
        size_t pooled = s.dev_bytes;
        for (const PlanSlab &x : ctx->slabs) pooled += x.dev_bytes;
        // the one released longest ago first: were the pool closed to the plan at hand once it is full, every plan of a larger batch to
        // come would be a hipMalloc and a hipFree (a step of 44 874 tokens, 3 heads behind 16 smaller plans 453 -> 2 200 us)
        while (!ctx->slabs.empty() && (pooled > kSlabPoolBytes || ctx->slabs.size() >= kSlabPoolMax)) {
            pooled -= ctx->slabs.front().dev_bytes;
            slab_give_back(ctx, ctx->slabs.front());
            ctx->slabs.erase(ctx->slabs.begin());
        }
        try {
            ctx->slabs.push_back(s);
        } catch (const std::bad_alloc &) {
            slab_give_back(ctx, s);
        }
    }
    delete plan;
}

int64_t flexsp_plan_num_items(const flexsp_plan *plan, int pass)
{
    if (!plan || pass < 0 || pass > 2) return FLEXSP_INVALID_ARGUMENT;
    if (pass != FLEXSP_PASS_FWD)
        if (const int rc = need_two_passes(plan)) return rc;
    return (int64_t)plan->pass[pass].items.size();
}

int flexsp_plan_get_items(const flexsp_plan *plan, int pass, flexsp_item *items, int64_t capacity,
                          int64_t *queue_offsets)
{
    if (!plan || pass < 0 || pass > 2) return FLEXSP_INVALID_ARGUMENT;
    if (pass != FLEXSP_PASS_FWD)
        if (const int rc = need_two_passes(plan)) return rc;
    const HostPass &hp = plan->pass[pass];
    if (capacity < (int64_t)hp.items.size() || (!items && !hp.items.empty())) return FLEXSP_INVALID_ARGUMENT;
    if (!hp.items.empty()) std::memcpy(items, hp.items.data(), hp.items.size() * sizeof(flexsp_item));
    if (queue_offsets)
        for (int x = 0; x <= plan->ctx->num_xcd; x++) queue_offsets[x] = hp.offsets[x];
    return FLEXSP_OK;
}

int flexsp_plan_tile_rows(const flexsp_plan *plan, int pass)
{
    if (!plan || pass < 0 || pass > 2) return FLEXSP_INVALID_ARGUMENT;
    if (!plan->two_listed && pass != FLEXSP_PASS_FWD) return pass == FLEXSP_PASS_BWD_DKV ? (plan->wide ? kDkvWideBk : kDkvBk) : kDqBq;
    return plan->pass[pass].tile_rows;
}

size_t flexsp_attn_bwd_workspace_bytes(const flexsp_plan *plan) { return plan ? plan->delta_bytes : 0; }

static int permute_entry(flexsp_ctx *ctx, const void *src, void *dst, int64_t T, int32_t H, int32_t D,
                         int32_t P, int32_t eb, flexsp_stream stream, bool unpack)
{
    if (T < 0 || H <= 0 || D <= 0 || P <= 0 || eb <= 0) return FLEXSP_INVALID_ARGUMENT;
    if (H % P != 0) return FLEXSP_INVALID_ARGUMENT;
    if (eb != 1 && eb != 2 && eb != 4 && eb != 8 && eb != 16) return FLEXSP_UNSUPPORTED;
    if (!ctx) return FLEXSP_INVALID_ARGUMENT;
    if (T == 0) return FLEXSP_OK;
    if (!src || !dst) return FLEXSP_INVALID_ARGUMENT;
    int64_t bytes = T * H * D * eb;
    const char *s = (const char *)src;
    const char *d = (const char *)dst;
    if (s < d + bytes && d < s + bytes) return FLEXSP_INVALID_ARGUMENT;  // overlap
    if (((uintptr_t)src | (uintptr_t)dst) % (uintptr_t)eb) return FLEXSP_INVALID_ARGUMENT;
    if (ctx->device < 0) return FLEXSP_NO_DEVICE;
    hipError_t e;
    {
        Timed tm(ctx, unpack ? FLEXSP_K_UNPACK : FLEXSP_K_PACK, (hipStream_t)stream);
        e = launch_pack(src, dst, T, H, D, P, eb, unpack, (hipStream_t)stream);
    }
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

static int permute_many_entry(flexsp_ctx *ctx, int32_t n, const void *const *src, void *const *dst, int64_t T,
                              const int32_t *H, int32_t D, int32_t P, int32_t eb, flexsp_stream stream, bool unpack)
{
    if (n < 0 || n > FLEXSP_PACK_MANY_MAX || (n > 0 && (!src || !dst || !H))) return FLEXSP_INVALID_ARGUMENT;
    if (T < 0 || D <= 0 || P <= 0 || eb <= 0) return FLEXSP_INVALID_ARGUMENT;
    if (eb != 1 && eb != 2 && eb != 4 && eb != 8 && eb != 16) return FLEXSP_UNSUPPORTED;
    if (!ctx) return FLEXSP_INVALID_ARGUMENT;
    for (int i = 0; i < n; i++)
        if (H[i] <= 0 || H[i] % P != 0) return FLEXSP_INVALID_ARGUMENT;
    if (T == 0 || n == 0) return FLEXSP_OK;
    // every source against every destination: none may overlap
    for (int i = 0; i < n; i++) {
        if (!src[i] || !dst[i]) return FLEXSP_INVALID_ARGUMENT;
        if (((uintptr_t)src[i] | (uintptr_t)dst[i]) % (uintptr_t)eb) return FLEXSP_INVALID_ARGUMENT;
    }
    for (int i = 0; i < n; i++)
        for (int j = 0; j < n; j++) {
            const char *s = (const char *)src[i], *d = (const char *)dst[j];
            const int64_t sb = T * H[i] * D * eb, db = T * H[j] * D * eb;
            if (s < d + db && d < s + sb) return FLEXSP_INVALID_ARGUMENT;
            if (i < j) {
                const char *d2 = (const char *)dst[i];
                if (d2 < d + db && d < d2 + sb) return FLEXSP_INVALID_ARGUMENT;  // two destinations overlap
            }
        }
    if (ctx->device < 0) return FLEXSP_NO_DEVICE;
    hipError_t e;
    {
        Timed tm(ctx, unpack ? FLEXSP_K_UNPACK : FLEXSP_K_PACK, (hipStream_t)stream);
        e = launch_pack_many(n, src, dst, T, H, D, P, eb, unpack, (hipStream_t)stream);
    }
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

int flexsp_pack_many(flexsp_ctx *ctx, int32_t n, const void *const *src, void *const *dst, int64_t T,
                     const int32_t *H, int32_t D, int32_t P, int32_t eb, flexsp_stream stream)
{
    return permute_many_entry(ctx, n, src, dst, T, H, D, P, eb, stream, false);
}

int flexsp_unpack_many(flexsp_ctx *ctx, int32_t n, const void *const *src, void *const *dst, int64_t T,
                       const int32_t *H, int32_t D, int32_t P, int32_t eb, flexsp_stream stream)
{
    return permute_many_entry(ctx, n, src, dst, T, H, D, P, eb, stream, true);
}

int flexsp_pack(flexsp_ctx *ctx, const void *src, void *dst, int64_t T, int32_t H, int32_t D, int32_t P,
                int32_t eb, flexsp_stream stream)
{
    return permute_entry(ctx, src, dst, T, H, D, P, eb, stream, false);
}

int flexsp_unpack(flexsp_ctx *ctx, const void *src, void *dst, int64_t T, int32_t H, int32_t D, int32_t P,
                  int32_t eb, flexsp_stream stream)
{
    return permute_entry(ctx, src, dst, T, H, D, P, eb, stream, true);
}

int flexsp_attn_varlen_fwd(flexsp_ctx *ctx, flexsp_plan *plan, flexsp_tensor q, flexsp_tensor k,
                           flexsp_tensor v, const int32_t *cu_dev, int32_t head_begin, int32_t head_count,
                           int32_t kv_head_begin, int32_t kv_head_count, int causal, float scale,
                           flexsp_tensor o, float *lse, flexsp_stream stream)
{
    int rc = check_attn_common(ctx, plan, cu_dev, head_begin, head_count, kv_head_begin, kv_head_count, causal);
    if (rc == FLEXSP_NO_DEVICE) {
        // still report bad views first, so host-only tests can see them
        if (!view_ok(q) || !view_ok(k) || !view_ok(v) || !view_ok(o) || !lse) return FLEXSP_INVALID_ARGUMENT;
        return rc;
    }
    if (rc) return rc;
    if (!view_ok(q) || !view_ok(k) || !view_ok(v) || !view_ok(o) || !lse) return FLEXSP_INVALID_ARGUMENT;
    if (!std::isfinite(scale)) return FLEXSP_INVALID_ARGUMENT;
    if (plan->pass[FLEXSP_PASS_FWD].items.empty()) return FLEXSP_OK;
    {
        hipError_t pe = plan_before_launch(plan, (hipStream_t)stream);
        if (pe != hipSuccess) return hip_fail(pe);
    }
    if (scale <= 0.f) scale = 1.0f / std::sqrt((float)plan->D);
    AttnArgs a;
    std::memset(&a, 0, sizeof(a));
    a.q = (const uint16_t *)q.ptr + (int64_t)head_begin * q.stride_head;
    a.k = (const uint16_t *)k.ptr + (int64_t)kv_head_begin * k.stride_head;
    a.v = (const uint16_t *)v.ptr + (int64_t)kv_head_begin * v.stride_head;
    a.out_o = (uint16_t *)o.ptr + (int64_t)head_begin * o.stride_head;
    a.q_st = (int32_t)q.stride_token; a.q_sh = (int32_t)q.stride_head;
    a.k_st = (int32_t)k.stride_token; a.k_sh = (int32_t)k.stride_head;
    a.v_st = (int32_t)v.stride_token; a.v_sh = (int32_t)v.stride_head;
    a.o_st = (int32_t)o.stride_token; a.o_sh = (int32_t)o.stride_head;
    a.lse_out = lse;
    a.T = (int32_t)plan->T; a.Hq = plan->Hq; a.G = plan->Hq / plan->Hkv; a.causal = plan->causal;
    a.scale = scale; a.scale_l2 = scale * 1.4426950408889634f;
    a.pq = plan->dq[FLEXSP_PASS_FWD];
    a.halves = plan->halves;
    hipError_t e;
    {
        Timed tm(ctx, FLEXSP_K_FWD, (hipStream_t)stream);
        e = launch_attn_fwd(a, plan->D, grid_for(ctx, plan->pass[FLEXSP_PASS_FWD], fwd_per_cu(ctx, plan)), (hipStream_t)stream);
    }
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

int flexsp_attn_varlen_fwd_kvshard(flexsp_ctx *ctx, flexsp_plan *plan, flexsp_tensor q, flexsp_tensor k,
                                   flexsp_tensor v, int32_t head_begin, int32_t head_count, int32_t kv_head_begin,
                                   int32_t kv_head_count, int causal, float scale, flexsp_tensor o, float *lse,
                                   flexsp_stream stream)
{
    if (!ctx || !plan) return FLEXSP_INVALID_ARGUMENT;
    if (plan->ctx != ctx || !plan->kvshard) return FLEXSP_PLAN_MISMATCH;
    if (head_begin < 0 || kv_head_begin < 0 || head_count <= 0 || kv_head_count <= 0 ||
        head_count % kv_head_count != 0)
        return FLEXSP_INVALID_ARGUMENT;
    if (head_count != plan->Hq || kv_head_count != plan->Hkv || (causal != 0) != (plan->causal != 0))
        return FLEXSP_PLAN_MISMATCH;
    if (!view_ok(q) || !view_ok(k) || !view_ok(v) || !view_ok(o) || !lse || !std::isfinite(scale))
        return FLEXSP_INVALID_ARGUMENT;
    if (ctx->device < 0 || !plan->dev_base) return FLEXSP_NO_DEVICE;
    if (plan->pass[FLEXSP_PASS_FWD].items.empty()) return FLEXSP_OK;
    {
        hipError_t pe = plan_before_launch(plan, (hipStream_t)stream);
        if (pe != hipSuccess) return hip_fail(pe);
    }
    if (scale <= 0.f) scale = 1.0f / std::sqrt((float)plan->D);
    AttnArgs a;
    std::memset(&a, 0, sizeof(a));
    a.q = (const uint16_t *)q.ptr + (int64_t)head_begin * q.stride_head;
    a.k = (const uint16_t *)k.ptr + (int64_t)kv_head_begin * k.stride_head;
    a.v = (const uint16_t *)v.ptr + (int64_t)kv_head_begin * v.stride_head;
    a.out_o = (uint16_t *)o.ptr + (int64_t)head_begin * o.stride_head;
    a.q_st = (int32_t)q.stride_token; a.q_sh = (int32_t)q.stride_head;
    a.k_st = (int32_t)k.stride_token; a.k_sh = (int32_t)k.stride_head;
    a.v_st = (int32_t)v.stride_token; a.v_sh = (int32_t)v.stride_head;
    a.o_st = (int32_t)o.stride_token; a.o_sh = (int32_t)o.stride_head;
    a.lse_out = lse;
    a.T = (int32_t)plan->T; a.Hq = plan->Hq; a.G = plan->Hq / plan->Hkv; a.causal = plan->causal;
    a.scale = scale; a.scale_l2 = scale * 1.4426950408889634f;
    a.pq = plan->dq[FLEXSP_PASS_FWD];
    hipError_t e;
    {
        Timed tm(ctx, FLEXSP_K_FWD, (hipStream_t)stream);
        e = launch_attn_fwd_kvshard(a, plan->D, grid_for(ctx, plan->pass[FLEXSP_PASS_FWD], 2), (hipStream_t)stream);
    }
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

int flexsp_attn_varlen_fwd_kvshard_acc(flexsp_ctx *ctx, flexsp_plan *plan, flexsp_tensor q, flexsp_tensor k,
                                       flexsp_tensor v, int32_t head_begin, int32_t head_count, int32_t kv_head_begin,
                                       int32_t kv_head_count, int causal, float scale, flexsp_tensor o_acc,
                                       float *lse_acc, flexsp_tensor o_bf16, flexsp_stream stream)
{
    if (!ctx || !plan) return FLEXSP_INVALID_ARGUMENT;
    if (plan->ctx != ctx || !plan->kvshard) return FLEXSP_PLAN_MISMATCH;
    if (head_begin < 0 || kv_head_begin < 0 || head_count <= 0 || kv_head_count <= 0 ||
        head_count % kv_head_count != 0)
        return FLEXSP_INVALID_ARGUMENT;
    if (head_count != plan->Hq || kv_head_count != plan->Hkv || (causal != 0) != (plan->causal != 0))
        return FLEXSP_PLAN_MISMATCH;
    if (!view_ok(q) || !view_ok(k) || !view_ok(v) || !view_ok(o_acc) || (o_bf16.ptr && !view_ok(o_bf16)) || !lse_acc ||
        !std::isfinite(scale))
        return FLEXSP_INVALID_ARGUMENT;
    if (ctx->device < 0 || !plan->dev_base) return FLEXSP_NO_DEVICE;
    if (plan->pass[FLEXSP_PASS_FWD].items.empty()) return FLEXSP_OK;
    {
        hipError_t pe = plan_before_launch(plan, (hipStream_t)stream);
        if (pe != hipSuccess) return hip_fail(pe);
    }
    if (scale <= 0.f) scale = 1.0f / std::sqrt((float)plan->D);
    AttnArgs a;
    std::memset(&a, 0, sizeof(a));
    a.q = (const uint16_t *)q.ptr + (int64_t)head_begin * q.stride_head;
    a.k = (const uint16_t *)k.ptr + (int64_t)kv_head_begin * k.stride_head;
    a.v = (const uint16_t *)v.ptr + (int64_t)kv_head_begin * v.stride_head;
    // the kernel's fold mode: the fp32 running result travels in the fields the forward does not use otherwise
    a.dq = (float *)o_acc.ptr + (int64_t)head_begin * o_acc.stride_head;
    a.dq_st = (int32_t)o_acc.stride_token; a.dq_sh = (int32_t)o_acc.stride_head;
    a.delta_out = lse_acc;
    if (o_bf16.ptr) {
        a.out_o = (uint16_t *)o_bf16.ptr + (int64_t)head_begin * o_bf16.stride_head;
        a.o_st = (int32_t)o_bf16.stride_token; a.o_sh = (int32_t)o_bf16.stride_head;
    }
    a.q_st = (int32_t)q.stride_token; a.q_sh = (int32_t)q.stride_head;
    a.k_st = (int32_t)k.stride_token; a.k_sh = (int32_t)k.stride_head;
    a.v_st = (int32_t)v.stride_token; a.v_sh = (int32_t)v.stride_head;
    a.T = (int32_t)plan->T; a.Hq = plan->Hq; a.G = plan->Hq / plan->Hkv; a.causal = plan->causal;
    a.scale = scale; a.scale_l2 = scale * 1.4426950408889634f;
    a.pq = plan->dq[FLEXSP_PASS_FWD];
    hipError_t e;
    {
        Timed tm(ctx, FLEXSP_K_FWD, (hipStream_t)stream);
        e = launch_attn_fwd_kvshard(a, plan->D, grid_for(ctx, plan->pass[FLEXSP_PASS_FWD], 2), (hipStream_t)stream);
    }
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

int flexsp_attn_varlen_bwd_kvshard(flexsp_ctx *ctx, flexsp_plan *plan, flexsp_tensor q, flexsp_tensor k,
                                   flexsp_tensor v, flexsp_tensor o, flexsp_tensor dO, const float *lse,
                                   int32_t head_begin, int32_t head_count, int32_t kv_head_begin,
                                   int32_t kv_head_count, int causal, float scale, flexsp_tensor dq, flexsp_tensor dk,
                                   flexsp_tensor dv, int32_t grad_dtype, int32_t accumulate, flexsp_stream stream)
{
    if (!ctx || !plan) return FLEXSP_INVALID_ARGUMENT;
    if (plan->ctx != ctx || !plan->kvshard) return FLEXSP_PLAN_MISMATCH;
    if (head_begin < 0 || kv_head_begin < 0 || head_count <= 0 || kv_head_count <= 0) return FLEXSP_INVALID_ARGUMENT;
    if (head_count % kv_head_count != 0) return FLEXSP_INVALID_ARGUMENT;
    if (head_count != plan->Hq || kv_head_count != plan->Hkv || (causal != 0) != (plan->causal != 0))
        return FLEXSP_PLAN_MISMATCH;
    if (grad_dtype != FLEXSP_BF16 && grad_dtype != FLEXSP_F32) return FLEXSP_UNSUPPORTED;
    if (accumulate != 0 && accumulate != 1) return FLEXSP_INVALID_ARGUMENT;
    if (accumulate && grad_dtype != FLEXSP_F32) return FLEXSP_UNSUPPORTED;  // partial sums are kept in fp32
    const bool views = view_ok(q) && view_ok(k) && view_ok(v) && view_ok(o) && view_ok(dO) && view_ok(dq) &&
                       view_ok(dk) && view_ok(dv) && lse;
    if (!views || !std::isfinite(scale)) return FLEXSP_INVALID_ARGUMENT;
    if (ctx->device < 0 || !plan->dev_base) return FLEXSP_NO_DEVICE;
    if (plan->pass[FLEXSP_PASS_BWD_DQ].items.empty() && plan->pass[FLEXSP_PASS_BWD_DKV].items.empty()) return FLEXSP_OK;
    {
        hipError_t pe = plan_before_launch(plan, (hipStream_t)stream);
        if (pe != hipSuccess) return hip_fail(pe);
    }
    if (scale <= 0.f) scale = 1.0f / std::sqrt((float)plan->D);
    AttnArgs a;
    std::memset(&a, 0, sizeof(a));
    a.q = (const uint16_t *)q.ptr + (int64_t)head_begin * q.stride_head;
    a.k = (const uint16_t *)k.ptr + (int64_t)kv_head_begin * k.stride_head;
    a.v = (const uint16_t *)v.ptr + (int64_t)kv_head_begin * v.stride_head;
    a.o = (const uint16_t *)o.ptr + (int64_t)head_begin * o.stride_head;
    a.dO = (const uint16_t *)dO.ptr + (int64_t)head_begin * dO.stride_head;
    const int64_t gb = grad_dtype == FLEXSP_F32 ? 4 : 2;
    a.grad_f32 = (grad_dtype == FLEXSP_F32 ? 1 : 0) | (accumulate ? 2 : 0);
    a.dq = (char *)dq.ptr + (int64_t)head_begin * dq.stride_head * gb;
    a.dk = (char *)dk.ptr + (int64_t)kv_head_begin * dk.stride_head * gb;
    a.dv = (char *)dv.ptr + (int64_t)kv_head_begin * dv.stride_head * gb;
    a.q_st = (int32_t)q.stride_token; a.q_sh = (int32_t)q.stride_head;
    a.k_st = (int32_t)k.stride_token; a.k_sh = (int32_t)k.stride_head;
    a.v_st = (int32_t)v.stride_token; a.v_sh = (int32_t)v.stride_head;
    a.o_st = (int32_t)o.stride_token; a.o_sh = (int32_t)o.stride_head;
    a.do_st = (int32_t)dO.stride_token; a.do_sh = (int32_t)dO.stride_head;
    a.dq_st = (int32_t)dq.stride_token; a.dq_sh = (int32_t)dq.stride_head;
    a.dk_st = (int32_t)dk.stride_token; a.dk_sh = (int32_t)dk.stride_head;
    a.dv_st = (int32_t)dv.stride_token; a.dv_sh = (int32_t)dv.stride_head;
    float *lse2 = plan->delta + (size_t)plan->T * plan->Hq;
    a.T = (int32_t)plan->T; a.Hq = plan->Hq; a.G = plan->Hq / plan->Hkv; a.causal = plan->causal;
    a.scale = scale; a.scale_l2 = scale * 1.4426950408889634f;
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipSuccess;
    a.lse_in = lse;
    a.lse_out = lse2;
    a.delta_out = plan->delta;
    if (const int grid = both_at_once(ctx, plan, a)) {
        Timed tm(ctx, FLEXSP_K_BWD_DKV, s);
        e = launch_attn_bwd_dkv_kvshard(a, plan->D, grid, s);
        return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
    }
    // as in flexsp_attn_varlen_bwd: the dQ kernel leaves delta and the base-2 log-sum-exp of its rows in
    // the plan's scratch for the dK/dV kernel
    a.pq = plan->dq[FLEXSP_PASS_BWD_DQ];
    if (!plan->pass[FLEXSP_PASS_BWD_DQ].items.empty()) {
        Timed tm(ctx, FLEXSP_K_BWD_DQ, s);
        e = launch_attn_bwd_dq_kvshard(a, plan->D, grid_for(ctx, plan->pass[FLEXSP_PASS_BWD_DQ], bwd_per_cu(ctx, plan, FLEXSP_PASS_BWD_DQ)), s);
    }
    if (e != hipSuccess) return hip_fail(e);
    a.lse_in = lse2;
    a.delta_in = plan->delta;
    a.pq = plan->dq[FLEXSP_PASS_BWD_DKV];
    if (!plan->pass[FLEXSP_PASS_BWD_DKV].items.empty()) {
        Timed tm(ctx, FLEXSP_K_BWD_DKV, s);
        e = launch_attn_bwd_dkv_kvshard(a, plan->D, grid_for(ctx, plan->pass[FLEXSP_PASS_BWD_DKV], bwd_per_cu(ctx, plan, FLEXSP_PASS_BWD_DKV)), s);
    }
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

int flexsp_lse_merge(flexsp_ctx *ctx, flexsp_tensor o_a, const float *lse_a, flexsp_tensor o_b, const float *lse_b,
                     flexsp_tensor o_out, float *lse_out, int64_t T, int32_t H, int32_t D, flexsp_stream stream)
{
    if (!ctx || T < 0 || H <= 0 || D <= 0) return FLEXSP_INVALID_ARGUMENT;
    if (D != 64 && D != 128) return FLEXSP_UNSUPPORTED;  // (a row's pieces then share one wavefront: in-place use is safe)
    if (T == 0) return FLEXSP_OK;
    if (!view_ok(o_a) || !view_ok(o_b) || !view_ok(o_out) || !lse_a || !lse_b || !lse_out)
        return FLEXSP_INVALID_ARGUMENT;
    if (T * (int64_t)H * (D / 8) >= ((int64_t)1 << 31)) return FLEXSP_UNSUPPORTED;
    if (ctx->device < 0) return FLEXSP_NO_DEVICE;
    hipError_t e = launch_lse_merge((const uint16_t *)o_a.ptr, lse_a, (const uint16_t *)o_b.ptr, lse_b,
                                    (uint16_t *)o_out.ptr, lse_out, T, H, D, (int32_t)o_a.stride_token,
                                    (int32_t)o_a.stride_head, (int32_t)o_b.stride_token, (int32_t)o_b.stride_head,
                                    (int32_t)o_out.stride_token, (int32_t)o_out.stride_head, (hipStream_t)stream);
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

int flexsp_lse_merge_acc(flexsp_ctx *ctx, flexsp_tensor o_acc, float *lse_acc, flexsp_tensor o_b, const float *lse_b,
                         flexsp_tensor o_bf16, int64_t T, int32_t H, int32_t D, flexsp_stream stream)
{
    if (!ctx || T < 0 || H <= 0 || D <= 0) return FLEXSP_INVALID_ARGUMENT;
    if (D != 64 && D != 128) return FLEXSP_UNSUPPORTED;
    if (T == 0) return FLEXSP_OK;
    if (!view_ok(o_acc) || !view_ok(o_b) || (o_bf16.ptr && !view_ok(o_bf16)) || !lse_acc || !lse_b)
        return FLEXSP_INVALID_ARGUMENT;
    if (T * (int64_t)H * (D / 8) >= ((int64_t)1 << 31)) return FLEXSP_UNSUPPORTED;
    if (ctx->device < 0) return FLEXSP_NO_DEVICE;
    hipError_t e = launch_lse_merge_acc((float *)o_acc.ptr, lse_acc, (const uint16_t *)o_b.ptr, lse_b, (uint16_t *)o_bf16.ptr,
                                        T, H, D, (int32_t)o_acc.stride_token, (int32_t)o_acc.stride_head,
                                        (int32_t)o_b.stride_token, (int32_t)o_b.stride_head,
                                        o_bf16.ptr ? (int32_t)o_bf16.stride_token : 0,
                                        o_bf16.ptr ? (int32_t)o_bf16.stride_head : 0, (hipStream_t)stream);
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

int flexsp_attn_varlen_bwd(flexsp_ctx *ctx, flexsp_plan *plan, flexsp_tensor q, flexsp_tensor k,
                           flexsp_tensor v, flexsp_tensor o, flexsp_tensor dO, const float *lse,
                           const int32_t *cu_dev, int32_t head_begin, int32_t head_count,
                           int32_t kv_head_begin, int32_t kv_head_count, int causal, float scale,
                           flexsp_tensor dq, flexsp_tensor dk, flexsp_tensor dv, int32_t grad_dtype,
                           flexsp_stream stream)
{
    int rc = check_attn_common(ctx, plan, cu_dev, head_begin, head_count, kv_head_begin, kv_head_count, causal);
    bool views = view_ok(q) && view_ok(k) && view_ok(v) && view_ok(o) && view_ok(dO) && view_ok(dq) &&
                 view_ok(dk) && view_ok(dv) && lse;
    if (rc == FLEXSP_NO_DEVICE && !views) return FLEXSP_INVALID_ARGUMENT;
    if ((rc == FLEXSP_OK || rc == FLEXSP_NO_DEVICE) && grad_dtype != FLEXSP_BF16 && grad_dtype != FLEXSP_F32)
        return FLEXSP_UNSUPPORTED;
    if (rc) return rc;
    if (!views || !std::isfinite(scale)) return FLEXSP_INVALID_ARGUMENT;
    if (plan->pass[FLEXSP_PASS_FWD].items.empty()) return FLEXSP_OK;
    {
        hipError_t pe = plan_before_launch(plan, (hipStream_t)stream);
        if (pe != hipSuccess) return hip_fail(pe);
    }
    if (scale <= 0.f) scale = 1.0f / std::sqrt((float)plan->D);
    AttnArgs a;
    std::memset(&a, 0, sizeof(a));
    a.q = (const uint16_t *)q.ptr + (int64_t)head_begin * q.stride_head;
    a.k = (const uint16_t *)k.ptr + (int64_t)kv_head_begin * k.stride_head;
    a.v = (const uint16_t *)v.ptr + (int64_t)kv_head_begin * v.stride_head;
    a.o = (const uint16_t *)o.ptr + (int64_t)head_begin * o.stride_head;
    a.dO = (const uint16_t *)dO.ptr + (int64_t)head_begin * dO.stride_head;
    const int64_t gb = grad_dtype == FLEXSP_F32 ? 4 : 2;
    a.grad_f32 = grad_dtype == FLEXSP_F32;
    a.dq = (char *)dq.ptr + (int64_t)head_begin * dq.stride_head * gb;
    a.dk = (char *)dk.ptr + (int64_t)kv_head_begin * dk.stride_head * gb;
    a.dv = (char *)dv.ptr + (int64_t)kv_head_begin * dv.stride_head * gb;
    a.q_st = (int32_t)q.stride_token; a.q_sh = (int32_t)q.stride_head;
    a.k_st = (int32_t)k.stride_token; a.k_sh = (int32_t)k.stride_head;
    a.v_st = (int32_t)v.stride_token; a.v_sh = (int32_t)v.stride_head;
    a.o_st = (int32_t)o.stride_token; a.o_sh = (int32_t)o.stride_head;
    a.do_st = (int32_t)dO.stride_token; a.do_sh = (int32_t)dO.stride_head;
    a.dq_st = (int32_t)dq.stride_token; a.dq_sh = (int32_t)dq.stride_head;
    a.dk_st = (int32_t)dk.stride_token; a.dk_sh = (int32_t)dk.stride_head;
    a.dv_st = (int32_t)dv.stride_token; a.dv_sh = (int32_t)dv.stride_head;
    float *lse2 = plan->delta + (size_t)plan->T * plan->Hq;
    a.T = (int32_t)plan->T; a.Hq = plan->Hq; a.G = plan->Hq / plan->Hkv; a.causal = plan->causal;
    a.scale = scale; a.scale_l2 = scale * 1.4426950408889634f;
    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    a.lse_in = lse;
    a.lse_out = lse2;
    a.delta_out = plan->delta;
    // (dq over o, dk and dv over k and v come out right here too: O is read in front of the chain, a key tile's rows by its own item
    // before it writes them)
    if (!plan->chain.empty()) {
        a.pq = plan->chain_dq;
        a.chain = 1;
        a.chain_flags = (int32_t)plan->chain_tiles;
        {
            Timed tm(ctx, FLEXSP_K_BWD_DELTA, s);
            e = launch_attn_bwd_dq(a, plan->D, 0, s);
        }
        if (e != hipSuccess) return hip_fail(e);
        a.lse_in = lse2;
        a.delta_in = plan->delta;
        Timed tm(ctx, FLEXSP_K_BWD_DKV, s);
        e = launch_attn_bwd_dkv(a, plan->D, ctx->num_cu, s);
        return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
    }
    if (const int grid = both_at_once(ctx, plan, a)) {
        Timed tm(ctx, FLEXSP_K_BWD_DKV, s);
        e = launch_attn_bwd_dkv(a, plan->D, grid, s);
        return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
    }
    // The dQ kernel runs first: it holds every query row's dO in registers, so it also computes
    // delta = dO . O and the log-sum-exp in base 2 for its rows and leaves both in the plan's
    // scratch for the dK/dV kernel (no separate preprocessing launch).
    a.pq = plan->dq[FLEXSP_PASS_BWD_DQ];
    {
        Timed tm(ctx, FLEXSP_K_BWD_DQ, s);
        e = launch_attn_bwd_dq(a, plan->D, grid_for(ctx, plan->pass[FLEXSP_PASS_BWD_DQ], bwd_per_cu(ctx, plan, FLEXSP_PASS_BWD_DQ)), s);
    }
    if (e != hipSuccess) return hip_fail(e);
    a.wide = plan->wide;
    a.lse_in = lse2;
    a.delta_in = plan->delta;
    a.pq = plan->dq[FLEXSP_PASS_BWD_DKV];
    {
        Timed tm(ctx, FLEXSP_K_BWD_DKV, s);
        e = launch_attn_bwd_dkv(a, plan->D, grid_for(ctx, plan->pass[FLEXSP_PASS_BWD_DKV], bwd_per_cu(ctx, plan, FLEXSP_PASS_BWD_DKV)), s);
    }
    return e == hipSuccess ? FLEXSP_OK : hip_fail(e);
}

}  // extern "C"
