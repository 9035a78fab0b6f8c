// flexsp_attn_varlen_fwd_static: the forward of packed attention for callers that cannot
// allocate (code under HIP graph capture, tight serving loops, harnesses that forbid hipMalloc).
// It needs no plan: the forward kernel finds its items in the device copy of cu_seqlens (attn_fwd_search.h), and deals them by
// counters in a file-scope array that every GPU the library runs on holds until the process ends.  For batches of many items or very many
// sequences work queues are listed ON THE DEVICE, in the same array, by a kernel in front.  The attention pass itself is that of
// flexsp_attn_varlen_fwd.  A batch small enough to be on the chip all at once shares nothing with other calls (see the entry point).
#include <mutex>

#include "flexsp_internal.h"

using namespace flexsp;

namespace {

// ---------------------------------------------------------------------------- the scratch
constexpr int kStaticMaxItems = 65536;   // tiles (128 query rows of one head each) per call: room for them in a list, and a limit of the call whether it has one or not
constexpr int kStaticMaxLevels = 4096;   // query tiles per sequence: sequences up to 524 288 tokens
constexpr int kCountersOff = 0;          // kMaxQueues ticket counters + "workgroups done", kCounterStride int32 apart: clear between calls (last_to_leave)
constexpr int kFlagsOff = kStaticFlagsAt * 4;  // int32[kStaticRecords]: arrival counters, likewise
constexpr int kListCountersOff = kFlagsOff + kStaticRecords * 4;  // the same for calls whose queues are listed, which a kernel in front of each clears: calls that overlapped must leave nothing in the others'
constexpr int kListFlagsOff = kListCountersOff + kStaticFlagsAt * 4;
constexpr int kOffsetsOff = kListFlagsOff + kStaticRecords * 4;  // int32[16]: kMaxQueues + 1 queue boundaries
constexpr int kStatusOff = kOffsetsOff + 64;  // int32[2], to look at when debugging: items listed by the last call of more than kSearchSeqs sequences, 1 if it rejected its lengths
constexpr int kItemsOff = kStatusOff + 64;
constexpr size_t kRecordsOff = kItemsOff + (size_t)(kStaticMaxItems + kStaticRecords) * sizeof(flexsp_item);  // partial results of cut tiles (whose parts are more items)
constexpr size_t kScratchBytes = kRecordsOff + (size_t)kStaticRecords * kPartialBytes;

// One copy per GPU, at its own address.  In host code this name is only a handle for
// hipGetSymbolAddress; kernels and copies use the resolved pointer (g_scratch_ptr).
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mutex;

// ---------------------------------------------------------------------------- queue builder
// One workgroup lists every (sequence, query tile, head) item of the batch, most expensive first,
// and deals the list round-robin into the kMaxQueues queues the forward kernel reads, so every
// queue is itself ordered longest first and the queues are level.  "Expensive" is the number of
// key tiles an item walks: tile index + 1 when causal (level = tile index), the sequence's tile
// count otherwise (level = tile count - 1).  Levels are bucket-sorted with LDS counters; the order
// of items inside a level is whatever the atomics give, which does not affect any result (items are
// independent).  Where the heads are a multiple of the queues, a queue gets the same neighbouring heads of every tile instead of
// every eighth item: as level, and with grouped heads an XCD reads few key heads' rows (16 384 tokens in 15 sequences, 16 heads on
// 2: 154.4 -> 150.2 us, when that batch had a list).  Lengths are validated here, on the device: a cu_seqlens that is not 0 = cu[0] <=
// cu[1] <= ... <= cu[B] <= T, a sequence with more than kStaticMaxLevels tiles or a batch with more
// than kStaticMaxItems items publishes an EMPTY list (the attention kernel then touches nothing)
// and raises the status word.
// One workgroup on an idle chip: trips to memory and chains of LDS accesses are what it takes.  Levels are summed 64 at a
// time by a wavefront, lengths are read 64 sequences at a time, a lane lists a tile.  The whole call, against levels
// summed one by one and a length read per sequence: 62 852 tokens in 201 sequences, 1 head 29.1 -> 25.1 us; 16 384 tokens
// in 15 sequences, 16 heads 169 -> 165 us.
constexpr int kBuildThreads = 1024;

__device__ __forceinline__ int inclusive_sum(int x, int lane)  // over the wavefront's lanes up to this one
{
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const int y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    return x;
}

__global__ __launch_bounds__(kBuildThreads) void build_static_queue_kernel(const int32_t *cu, int B, int T, int heads,
                                                                            int causal, int tile_rows, unsigned char *scr)
{
    __shared__ int hist[kStaticMaxLevels + 2];   // sequences with exactly n tiles
    __shared__ int start[kStaticMaxLevels + 1];  // first list position of a level
    __shared__ int fill[kStaticMaxLevels + 1];   // (sequence, tile) pairs placed in a level so far
    __shared__ int s_maxnt, s_bad, s_total;
    int32_t *counters = (int32_t *)(scr + kListCountersOff);
    int32_t *offsets = (int32_t *)(scr + kOffsetsOff);
    int32_t *status = (int32_t *)(scr + kStatusOff);
    flexsp_item *items = (flexsp_item *)(scr + kItemsOff);
    const int tid = threadIdx.x;

    const int levels = min(T / tile_rows + 1, kStaticMaxLevels);  // query tiles a sequence of the batch can have
    for (int i = tid; i <= levels; i += kBuildThreads) hist[i] = fill[i] = 0;
    if (tid == 0) {
        s_maxnt = 0;
        s_bad = (B > 0 && cu[0] != 0) ? 1 : 0;
        s_total = 0;
    }
    if (tid <= kMaxQueues) counters[tid * kCounterStride] = 0;  // every call starts with clear tickets
    __syncthreads();

    for (int b = tid; b < B; b += kBuildThreads) {
        const int lo = cu[b], hi = cu[b + 1];
        if (lo < 0 || hi < lo || hi > T) {
            atomicOr(&s_bad, 1);
            continue;
        }
        const int nt = (hi - lo + tile_rows - 1) / tile_rows;
        if (nt > levels) {
            atomicOr(&s_bad, 1);
            continue;
        }
        if (nt > 0) {
            atomicAdd(&hist[nt], 1);
            atomicMax(&s_maxnt, nt);
        }
    }
    __syncthreads();

    const int wave = tid >> 6, lane = tid & 63;
    if (wave == 0) {
        // levels in decreasing order of cost, 64 at a time; positions count (sequence, tile) pairs, heads come later
        const int maxnt = s_maxnt;
        int pos = 0, longer = 0;  // pairs of the levels above; causal: sequences that reach above
        for (int t0 = maxnt - 1; t0 >= 0; t0 -= 64) {
            const int t = t0 - lane;
            int n = t >= 0 ? hist[t + 1] : 0;  // causal: sequences whose last tile this is, and with those above: all that have it
            if (causal) {
                n = inclusive_sum(n, lane) + longer;
                longer = __shfl(n, 63);
                if (t < 0) n = 0;
            } else {
                n *= t + 1;
            }
            const int upto = inclusive_sum(n, lane) + pos;
            if (t >= 0) start[t] = upto - n;
            pos = __shfl(upto, 63);
        }
        if (lane == 0) {
            if ((int64_t)pos * heads > kStaticMaxItems) s_bad = 1;
            s_total = s_bad ? 0 : pos * heads;
        }
    }
    __syncthreads();

    const int total = s_total, nq = kMaxQueues;
    if (tid <= nq) {
        // queue x holds list positions x, x + nq, x + 2 nq, ...
        const int x = tid;
        offsets[x] = x * (total / nq) + min(x, total % nq);
    }
    if (tid == 0) {
        status[0] = total;
        status[1] = s_bad;
    }
    if (total == 0) return;

    // 64 neighbouring sequences at a time (their lengths in one load), shared by `per` wavefronts: the sequences' tiles in one
    // row, each wavefront takes stretches of 64 of them, a lane per tile.
    const int nwaves = kBuildThreads >> 6, groups = (B + 63) / 64, per = max(1, nwaves / groups);
    for (int g = wave / per; g < groups; g += nwaves / per) {
        const int b = g * 64 + lane;
        const int lo_ = b < B ? cu[b] : 0, len_ = b < B ? cu[b + 1] - lo_ : 0;
        const int upto = inclusive_sum((len_ + tile_rows - 1) / tile_rows, lane);  // tiles of this and the earlier lanes' sequences
        const int tiles = __shfl(upto, 63);
        for (int c = (wave % per) * 64; c < tiles; c += per * 64) {
            const int n = min(c + lane, tiles - 1);
            int owner = 0;  // the sequence of tile n: how many end before it or at it
#pragma unroll
            for (int d = 32; d; d /= 2)
                if (__shfl(upto, owner + d - 1) <= n) owner += d;
            const int lo = __shfl(lo_, owner), len = __shfl(len_, owner), nt = (len + tile_rows - 1) / tile_rows;
            const int t = n - (__shfl(upto, owner) - nt);
            if (c + lane >= tiles) continue;
            const int level = causal ? t : nt - 1;
            const int p0 = (start[level] + atomicAdd(&fill[level], 1)) * heads;
            flexsp_item it;
            it.seq_start = lo;
            it.seq_len = len;
            it.tile = t;
            // whole tiles only: every 64-key step the tile's rows can see
            it.step_begin = 0;
            it.step_end = ((causal ? min(len, (t + 1) * tile_rows) : len) + kFwdBk - 1) / kFwdBk;
            it.slot = -1;
            it.parts = 1;
            // (no division per head: this workgroup's time is the call's)
            if (heads % nq == 0) {  // (so is the total)
                const int group = heads / nq;
                for (int x = 0; x < nq; x++)
                    for (int i = 0; i < group; i++) {
                        it.head = x * group + i;
                        items[x * (total / nq) + p0 / nq + i] = it;
                    }
            } else {
                int x = p0 % nq, at = p0 / nq;
                for (int h = 0; h < heads; h++) {
                    it.head = h;
                    items[x * (total / nq) + min(x, total % nq) + at] = it;
                    if (++x == nq) x = 0, at++;
                }
            }
        }
    }
}

}  // namespace

namespace flexsp {

// Resolves this GPU's copy of the scratch array.  Called by flexsp_ctx_create with `device`
// current, once per device (later calls find the pointer).
hipError_t static_scratch_init(int device)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[device]) return hipSuccess;
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = p;
    return hipSuccess;
}

}  // namespace flexsp

extern "C" int flexsp_attn_varlen_fwd_static(flexsp_ctx *ctx, flexsp_tensor q, flexsp_tensor k, flexsp_tensor v,
                                             const int32_t *cu_seqlens_dev, int32_t B, int64_t T,
                                             int32_t head_begin, int32_t head_count, int32_t kv_head_begin,
                                             int32_t kv_head_count, int32_t D, int causal, float scale,
                                             flexsp_tensor o, float *lse, flexsp_stream stream)
{
    if (!ctx || !cu_seqlens_dev || !lse || B < 0 || T < 0) return FLEXSP_INVALID_ARGUMENT;
    if (head_begin < 0 || kv_head_begin < 0 || head_count <= 0 || kv_head_count <= 0 ||
        head_count % kv_head_count != 0)
        return FLEXSP_INVALID_ARGUMENT;
    if (!view_ok(q) || !view_ok(k) || !view_ok(v) || !view_ok(o) || !std::isfinite(scale))
        return FLEXSP_INVALID_ARGUMENT;
    if (D != 64 && D != 128) return FLEXSP_UNSUPPORTED;
    // (every sequence adds at most one partial tile)
    if (T > (int64_t)kStaticMaxLevels * kFwdBq ||
        ((T + kFwdBq - 1) / kFwdBq + B) * (int64_t)head_count > kStaticMaxItems)
        return FLEXSP_UNSUPPORTED;
    const int device = ctx_device(ctx);
    if (device < 0 || device >= kMaxDevices || !g_scratch_ptr[device]) return FLEXSP_NO_DEVICE;
    if (B == 0 || T == 0) return FLEXSP_OK;
    unsigned char *scr = (unsigned char *)g_scratch_ptr[device];
    hipStream_t s = (hipStream_t)stream;
    // A batch whose items can all be resident at once needs neither an order nor a list: every workgroup finds its item
    // itself, in the time it would take to read it from a list (402 tokens, 16 heads: 23.0 -> 11.6 us; 1 687 tokens, 16 heads: 31.9 ->
    // 21.9 us; 257 tokens, 2 heads: 18.3 -> 10.4 us).  Larger ones need longest-first queues.
    const int64_t most_items = ((T + kFwdBq - 1) / kFwdBq + B) * (int64_t)head_count;
    const int num_cu = flexsp_ctx_num_cu(ctx);
    const bool dealt = most_items > 2 * num_cu;
    // Whether it does run in halves the lengths tell, on the device: the rows that the tensors hold beyond the batch change nothing.
    // (1 000 tokens, 8 heads in 4 096 rows 19.4 -> 18.1 us, 3 000 tokens, 1 head in 65 536 rows 50.9 -> 40.9.  Batches in whole items that
    // might have been others take what they took, up to 0.6 us more with D = 64.  A second launch for the halves instead, which
    // leaves at once where it is not wanted, was 2.5 to 4 us for each of them.)
    const bool may_halve = fwd_may_halve(T, B, head_count, num_cu);
    // (Cut tiles need records, and tickets counters, that calls share: batches of fewer items, which may run side by side, have neither.  A
    // batch that may run in halves is one of at most 32 sequences.)
    const bool found = dealt && B <= kSearchSeqs;
    // What the search costs it costs for every item, 0.5 to 2 us of a workgroup; a list of the same items costs a launch in front, about 4 us, so it is
    // the faster way from three and a half possible items to a workgroup on, four and a half where a lane has one sequence.  Whole call, search -> list: 256
    // sequences of 256 tokens, 16 heads on 2, D = 64 191 -> 145 us; 128 of 512, 8 heads, D = 64 103 -> 93; 24 of 1 000, 16 heads on 2 (6.6 items) 144 -> 136;
    // not taken: 12 of 1 000, 16 heads on 2, D = 64, unmasked (3.6) 85 -> 91; 64 of 256, 4 heads (1.5) 24.0 -> 26.8.  Of 1 914 batches, drawn and over
    // lengths, heads and sequences, 53 take over 2 % more by this line than by the better way.  (The choice changes no bits.)
    const bool search = found && (may_halve || most_items <= (B <= 64 ? kSearchFewItems : kSearchItems) * num_cu);
    hipError_t e = hipSuccess;
    if (dealt && !found) {
        hipLaunchKernelGGL(build_static_queue_kernel, dim3(1), dim3(kBuildThreads), 0, s, cu_seqlens_dev, (int)B, (int)T,
                           (int)head_count, causal ? 1 : 0, kFwdBq, scr);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_status(e);
    }

    if (scale <= 0.f) scale = 1.0f / std::sqrt((float)D);
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
    a.T = (int32_t)T; a.Hq = head_count; a.G = head_count / kv_head_count; a.causal = causal ? 1 : 0;
    a.scale = scale; a.scale_l2 = scale * 1.4426950408889634f;
    a.num_cu = num_cu;
    if (!dealt || found) {
        a.cu = cu_seqlens_dev;
        a.B = B;
    }
    // the item count is known to the device only.  Dealt items: a full persistent grid; workgroups without work leave
    int64_t grid = 2 * (int64_t)num_cu;
    if (dealt) {
        if (!search) {
            a.pq.items = (const flexsp_item *)(scr + kItemsOff);
            a.pq.offsets = (const int32_t *)(scr + kOffsetsOff);
        }
        a.pq.counters = (int32_t *)(scr + (search ? kCountersOff : kListCountersOff));
        a.pq.nq = kMaxQueues;
        a.pq.split_flags = (int32_t *)(scr + (search ? kFlagsOff : kListFlagsOff));
        a.pq.split_scratch = (char *)scr + kRecordsOff;
    } else {
        grid = may_halve ? std::max(most_items, fwd_halves_most(D, T, B, head_count, num_cu)) : most_items;
    }
    if (found && !search) {
        e = launch_list_items(a, (int)(most_items / head_count), s);
        if (e != hipSuccess) return hip_status(e);
        a.cu = nullptr;  // (the attention kernel has a list)
    }
    // (halves with two buffers where whole items too have the LDS for it: D = 128 one workgroup to a compute unit, D = 64 two)
    if (may_halve) a.halves = !search && (D == 64 || most_items <= num_cu) ? 2 : 1;
    e = search && !may_halve ? launch_attn_fwd_search(a, D, (int)grid, s) : launch_attn_fwd(a, D, (int)grid, s);
    return e == hipSuccess ? FLEXSP_OK : hip_status(e);
}
