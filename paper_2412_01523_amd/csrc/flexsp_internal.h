// Internal declarations shared by the host code and the kernels of libflexsp.
// Nothing here is part of the public ABI (see include/flexsp.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>
#include <cstring>

#include "flexsp.h"

namespace flexsp {

// Tile shapes.  The plan builder and the kernels must agree on these.
constexpr int kFwdBq = 128;    // query rows per forward work item (4 waves x 32 rows)
constexpr int kFwdBk = 64;     // key rows staged in LDS per forward step
constexpr int kDqBq = 128;     // query rows per dQ work item
constexpr int kDqBk = 64;      // key rows per dQ step
constexpr int kDkvBk = 64;     // key rows per dK/dV work item (2 pairs of waves x 32 rows)
constexpr int kDkvWideBk = 128;  // ... of attn_bwd_dkv_wide_kernel's (4 waves x 32 rows)
constexpr int kDkvBq = 64;     // query rows per dK/dV step
constexpr int kChainBk = 128;  // key rows per item of a backward in one pass (8 waves: 4 blocks of 32 rows, dK and dV apart)
constexpr int kThreads = 256;  // every attention kernel runs 4 wavefronts per workgroup
constexpr int kMaxQueues = 8;  // one work queue per XCD
constexpr int kCounterStride = 32;  // int32 from one queue's ticket counter to the next: a 128-byte line each
constexpr int kLateTicketSteps = 16;  // items of at least this many steps draw the next ticket near their end

// Split tiles (see flexsp_item in flexsp.h): a part's partial result is one record of fp32 values,
// 64 per thread of the workgroup (the accumulators) plus, for the forward, each row's running
// maximum and sum.  kMinPartSteps: no part is made shorter than this many inner-loop steps (the
// hand-over costs about as much as two or three steps); at most kMaxParts parts per tile and
// kMaxSplitRecords records per pass.
constexpr int kPartialBytes = 64 * kThreads * 4 + 2 * kThreads * 4;  // 67 584 B
constexpr int kMinPartSteps = 16;
constexpr int kShortPartSteps = 4;  // ... where a backward would leave compute units without work (see direct_list)
constexpr int kGroupMajorSteps = 24;  // sequences whose longest tile has at most this many steps are queued tile beside tile
constexpr int kLongPartSteps = 160;  // parts at least this long are aimed at 35 % of an even share instead of 75 %
constexpr int kMaxParts = 8;
constexpr int64_t kPartAffinityBytes = (int64_t)7 << 19;  // 3.5 MiB of an XCD's 4 MiB of L2 (see split_long_items)
constexpr int kSplitSteps = 4;  // a forward in halves (attn_fwd_kernel) splits walks of at least this many steps
constexpr int kMaxSplitRecords = 2048;
constexpr int kSearchSeqs = 256;      // a forward without a plan finds its items in the lengths of up to so many sequences (attn_fwd_search.hip), four to a lane in registers
constexpr int kSearchItems = 7;       // ... each workgroup by itself, up to so many items per compute unit; of more a kernel in front makes a list
constexpr int kSearchFewItems = 9;    // ... with at most 64 sequences, a lane each
// ... and has so many partial-result records.  Parts are 0.35 to 0.75 even shares, so up to some 750 in all suffice unless a few heads' long tiles are
// cut at 0.35 shares and 160 steps: of 7 440 drawn batches 249 have cut tiles, half of those need 600 records, nine in ten 726, seven over 1 024 (up to 1 650).  Those are
// cut into fewer parts (SearchBatch); 512 would do for 75.
constexpr int kStaticRecords = 1024;
constexpr int kStaticFlagsAt = (kMaxQueues + 1) * kCounterStride;  // ... whose arrival counters stand so many int32 behind its ticket counters

// One workgroup's leave from a launch whose counters calls without a plan share: true for the one that has to clear them.  Such calls have
// to be ordered, but if two overlap all the same nothing of it may stay for the calls after them, which have no plan of their own to
// start from.  So leaves are never overwritten: they are counted over all launches (of one grid size each) and taken off by the
// `grid`, however those mix, and once every workgroup of all of them has left, the count is 0 and the last one has cleared what they drew and
// counted.  (A count set to 0 by whoever finds the others there lost the leaves that came in between.)  WORD: add(n) returns the
// value before.
template <class WORD>
__host__ __device__ inline bool last_to_leave(WORD &&left, unsigned grid)
{
    const unsigned n = left.add(1u) + 1u;
    if (n < grid || (n > grid && n % grid)) return false;
    left.add(0u - grid);
    return true;
}

// A backward in one pass (attn_bwd_chain.hip, build_chain).
constexpr int kChainDies = 16;   // compute dies, each of which draws from a word of its own
constexpr int kChainTeam = 32;   // a long sequence's key tiles are bundles of up to so many, a workgroup of the die each
constexpr int kChainSpan = 64;   // shorter ones are put together until a bundle has so many items
constexpr size_t kChainTileBytes = (size_t)kDkvBq * 128 * sizeof(float);        // partial sums of dQ: 64 query rows of a head, D = 128
constexpr int64_t kChainMostTiles = ((int64_t)4 << 30) / (int64_t)kChainTileBytes;  // a plan keeps up to 4 GiB of them

// How a chain's workgroups get their items.  The list is cut into bundles (build_chain).  A compute die takes a bundle at a time, in the order of the
// list, and its workgroups draw the bundle's items one by one: what a bundle shares meets in the die's L2.  A die's word holds the next item and the end
// of its bundle (end << 32 | next); whoever draws the item at the end takes the next bundle for the die, the others wait for that.  Returns the
// item that a draw of the word's value `w` stands for, or -1 when there are no more.
// Every wait ends, however few workgroups are resident.  An item waits for items in front of it in the list only.  Of all items that are not
// done, take the first: what it waits for is done.  If it has been drawn, a running workgroup has it, and finishes it.  If not, but its
// bundle has been taken, the workgroups of that die have drawn only from what stands in front of it (a die takes a bundle when the one
// before has been drawn to the end), all of it done, so they are free and draw it; there is such a workgroup, for whoever takes a
// bundle draws from it.  If its bundle has not been taken, neither has any behind it: everybody who runs is free, or holds something that is
// done, and takes it.  A workgroup that waits for a bundle to be taken waits for one that waits for nobody.
// DIE: draw() adds one to the word and returns what it was, look() reads it, put(w) replaces it, bundle() counts bundles taken (of all dies), low(w) and
// high(w) are a word's halves, rest() passes some time.
constexpr uint32_t kChainDone = 0x80000000u;
template <class DIE>
__host__ __device__ __forceinline__ int chain_take(DIE &&die, unsigned long long w, const int32_t *offsets, int bundles)
{
    for (;;) {
        const uint32_t at = die.low(w), end = die.high(w);
        if (at & kChainDone) return -1;
        if (at < end) return (int)at;
        if (at == end) {
            const uint32_t b = die.bundle();
            const bool more = b < (uint32_t)bundles;
            const uint32_t first = more ? (uint32_t)offsets[b] : 0, stop = more ? (uint32_t)offsets[b + 1] : 0;
            die.put(more ? (unsigned long long)stop << 32 | (first + 1) : (unsigned long long)kChainDone);
            return more ? (int)first : -1;
        }
        for (;;) {
            const unsigned long long v = die.look();
            if (die.high(v) != end || (die.low(v) & kChainDone)) break;
            die.rest();
        }
        w = die.draw();
    }
}

// Work item of the key-shard forward: query rows q_start .. q_start+q_len-1 of q / o / lse, shard
// keys k_start .. k_start+k_len-1 of k / v, shift = position of the first query in its sequence
// minus position of the shard's first key.  `tile` counts 128-row query tiles.
// A tile cut into parts (see flexsp_item) is listed once per part, each with its own key range and the
// shift that goes with it: head_parts = head | part << 16 | nparts << 24 (0 and 1 for a whole tile),
// slot = the tile's first partial-result record (-1 for a whole tile).
struct flexsp_shard_item {
    int32_t q_start, q_len, k_start, k_len, shift, tile, head_parts, slot;
};

struct PassQueues {
    const flexsp_item *items;  // device, all queues back to back
    const int32_t *offsets;    // device, nq + 1 boundaries into items
    int32_t *counters;         // device, nq fetch counters + 1 "workgroups done" counter, kCounterStride apart
    int32_t nq;
    int32_t *split_flags;      // device, one arrival counter per partial-result record (a tile uses its first record's)
    char *split_scratch;       // device, kPartialBytes per record
    int32_t direct;            // the launch has one workgroup per item: workgroup w runs items[w] and leaves (see ItemDealer)
};

// Arguments of the attention kernels.  Strides are in elements; pointers already include
// the first head of the subset.
struct AttnArgs {
    const uint16_t *q, *k, *v, *o, *dO;
    uint16_t *out_o;
    void *dq, *dk, *dv;  // bf16 or fp32 elements, see grad_f32
    const float *lse_in, *delta_in;
    float *lse_out, *delta_out;
    // strides in elements; 32-bit (checked by the host) to keep the kernels' scalar registers free
    int32_t q_st, q_sh, k_st, k_sh, v_st, v_sh, o_st, o_sh, do_st, do_sh;
    int32_t dq_st, dq_sh, dk_st, dk_sh, dv_st, dv_sh;
    int32_t T;       // tokens in the packed stream (row length of lse / delta)
    int32_t Hq;      // query heads in the subset
    int32_t G;       // query heads per kv head
    int32_t causal;
    int32_t grad_f32;  // bit 0: gradients are stored as fp32 instead of bf16; bit 1 (key-shard kernels): added to what is there
    float scale;     // softmax scale
    float scale_l2;  // scale * log2(e)
    PassQueues pq;
    // a launch that runs both backward passes (launch_attn_bwd_dkv*, both passes direct, lse_in as the caller gave it): the
    // dQ pass's queues, its first workgroup (0: the dK/dV pass alone), the dK/dV pass's items
    PassQueues dq_pq;
    int32_t dq_wg, dkv_items;
    int32_t wide;  // the dK/dV pass's items have kDkvWideBk keys
    int32_t grid;  // workgroups of the launch (filled in by the launchers)
    // a forward without a plan: the lengths (device), in which every workgroup finds its item unless pq holds a list
    const int32_t *cu;
    int32_t B;
    // a forward in halves: pq lists tiles of kHalfBq query rows; with cu: in halves if the lengths say so (attn_fwd_either_kernel, with that
    // many buffers)
    int32_t halves;
    int32_t num_cu;  // (for that decision)
    // a backward in one pass (the dQ launcher then starts what runs in front of it); its flags, which that clears
    int32_t chain, chain_flags;
};

// Launchers implemented next to their kernels.  All are asynchronous on `s`.
hipError_t launch_pack(const void *src, void *dst, int64_t T, int H, int D, int P, int eb,
                       bool unpack, hipStream_t s);
hipError_t launch_pack_many(int n, const void *const *src, void *const *dst, int64_t T, const int32_t *H, int D,
                            int P, int eb, bool unpack, hipStream_t s);
hipError_t launch_attn_fwd(const AttnArgs &a, int D, int grid, hipStream_t s);
hipError_t launch_attn_fwd_search(const AttnArgs &a, int D, int grid, hipStream_t s);  // a.cu, a.pq.counters, split_flags and split_scratch: no list
hipError_t launch_list_items(const AttnArgs &a, int positions, hipStream_t s);  // ... which this writes: a.pq.items, offsets, and clear counters and split_flags; positions: wavefronts
hipError_t launch_attn_fwd_kvshard(const AttnArgs &a, int D, int grid, hipStream_t s);  // a.pq.items: flexsp_shard_item
hipError_t launch_lse_merge(const uint16_t *oa, const float *la, const uint16_t *ob, const float *lb, uint16_t *oo,
                            float *lo, int64_t T, int H, int D, int32_t oa_st, int32_t oa_sh, int32_t ob_st,
                            int32_t ob_sh, int32_t oo_st, int32_t oo_sh, hipStream_t s);
hipError_t launch_lse_merge_acc(float *oacc, float *lacc, const uint16_t *ob, const float *lb, uint16_t *ob16, int64_t T,
                                int H, int D, int32_t oa_st, int32_t oa_sh, int32_t ob_st, int32_t ob_sh, int32_t o16_st,
                                int32_t o16_sh, hipStream_t s);
hipError_t launch_attn_bwd_dkv(const AttnArgs &a, int D, int grid, hipStream_t s);
hipError_t launch_attn_bwd_dq(const AttnArgs &a, int D, int grid, hipStream_t s);
hipError_t launch_attn_bwd_delta(const AttnArgs &a, hipStream_t s);
hipError_t launch_attn_bwd_chain(const AttnArgs &a, int grid, hipStream_t s);
hipError_t launch_attn_bwd_dkv_kvshard(const AttnArgs &a, int D, int grid, hipStream_t s);  // a.pq.items: flexsp_shard_item;
hipError_t launch_attn_bwd_dq_kvshard(const AttnArgs &a, int D, int grid, hipStream_t s);   // a.grad_f32 bit 1: add to dq / dk / dv

// Whether a forward of whole tiles runs in halves (see attn_fwd.hip).  Decided from what the batch itself holds: tokens, sequences, tiles
// of 64 query rows (kHalfBq) over all heads, their key tiles, and the tiles of the longest sequence.  The plan and a launch without one
// (on the device: attn_fwd_either_kernel) then agree whatever the tensors have room for, and a batch whose tiles the plan does not
// cut has the same bits with and without a plan.
// A walk has to be worth a hand-over (512 tokens a sequence), and all tiles at work at once, one per compute unit: a second turn costs
// what the halves save.  Where a long sequence's tiles outlast the rest, more of them find room meanwhile: up to a third more tiles
// with D = 128, three to a unit with D = 64, if all their steps are no more than the units take (D = 128: four fifths; D = 64, whose two
// workgroups fill each other's waits, five quarters beside 5 120 tokens) while the
// longest tile lasts whole.
// Forward without a plan, whole items -> halves, one sequence: 512 tokens, 8 heads 13.0 -> 11.7 us; 1 024, 8 heads 19.3 -> 15.6; 3 000, 4
// heads 40.8 -> 28.3; 5 248, 4 heads 68.0 -> 56.2; not causal 2 000, 8 heads 32.9 -> 26.4; D = 64: 700, 2 heads 11.1 -> 10.4; 4 000, 4 heads
// 38.6 -> 26.6; four sequences, one of 15 911, 1 head, not causal 153 -> 95; 261 drawn batches 1.01 to 1.76 times as fast, 1.32 on average.
// Beyond the lines (in a build whose halves took 5 % longer): not causal 2 176, 8 heads 32.6 -> 46.9; 1 152, 16 heads 20.6 -> 31.9, causal
// 20.7 -> 24.2; 5 248, 4 heads 73 -> 93; D = 64: 3 600, 8 heads, not causal 37.8 -> 43.1.
inline constexpr int kHalfBq = 64;
struct HalvesCount {
    int64_t tokens, seqs, tiles, steps, longest;
};
__host__ __device__ inline int fwd_halves_room(int D, int num_cu) { return D == 128 ? 4 * num_cu / 3 : 3 * num_cu; }
__host__ __device__ inline bool fwd_halves(int D, const HalvesCount &c, int num_cu)
{
    if (c.tokens < 512 * c.seqs || c.tiles > fwd_halves_room(D, num_cu)) return false;
    if (c.tiles <= num_cu) return true;
    const int64_t while_longest = c.longest * num_cu;
    return c.longest >= 32 && (D == 128 ? 5 * c.steps <= 4 * while_longest : 4 * c.steps <= (c.longest >= 80 ? 5 : 4) * while_longest);
}
// Whether any batch of B sequences and at most T tokens may run in halves (512 tokens, 8 tiles, to a sequence).
inline bool fwd_may_halve(int64_t T, int64_t B, int64_t heads, int num_cu) { return T >= 512 * B && 8 * B * heads <= num_cu; }
// ... and the most workgroups it then has.
inline int64_t fwd_halves_most(int D, int64_t T, int64_t B, int64_t heads, int num_cu)
{
    const int64_t all = ((T + kHalfBq - 1) / kHalfBq + B) * heads, room = fwd_halves_room(D, num_cu);
    return all < room ? all : room;
}

// Host helpers shared by the files that hold entry points.
int ctx_device(const flexsp_ctx *ctx);        // HIP device of a context, -1 for a host-only one
int hip_status(hipError_t e);                 // records e for flexsp_last_hip_error, returns the flexsp_status for it
hipError_t static_scratch_init(int device);   // resolves the device's copy of the no-allocation scratch array

// A view the attention kernels can address: 16-byte aligned rows, strides that fit the kernels'
// 32-bit arithmetic (a per-lane byte offset spans up to 64 token rows).
inline bool view_ok(const flexsp_tensor &t)
{
    if (!t.ptr) return false;
    if (((uintptr_t)t.ptr & 15) != 0) return false;
    if (t.stride_token <= 0 || t.stride_head <= 0) return false;
    if ((t.stride_token % 8) != 0 || (t.stride_head % 8) != 0) return false;
    if (t.stride_token > (1 << 24) || t.stride_head > 0x3fffffff) return false;
    return true;
}

}  // namespace flexsp
