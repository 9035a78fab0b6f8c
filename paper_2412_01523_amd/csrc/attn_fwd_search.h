// Items of a forward without a plan, found in the lengths.
#pragma once

#include "attn_fwd_pass.h"

namespace flexsp {
namespace {

// Sum and maximum over the wavefront's lanes: rows of 16 by cross-lane operands, then the four rows as scalars.
template <int CTRL>
__device__ __forceinline__ int dpp(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true); }
__device__ __forceinline__ int lanes_sum(int x)
{
    x += dpp<0xB1>(x);
    x += dpp<0x4E>(x);
    x += dpp<0x141>(x);
    x += dpp<0x140>(x);
    return __builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16) + __builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48);
}
__device__ __forceinline__ int lanes_max(int x)
{
    x = max(x, dpp<0xB1>(x));
    x = max(x, dpp<0x4E>(x));
    x = max(x, dpp<0x141>(x));
    x = max(x, dpp<0x140>(x));
    return max(max(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               max(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

// The list that a small kernel in front of this one would write (build_static_queue_kernel), without writing it: items in decreasing order of the key tiles
// their query tile walks, which a level stands for (the tile's number if causal, else the sequence's number of tiles less one),
// levels from the highest down.  A place in it is found by halving over the levels, with the lengths in the lanes, 64 sequences at a
// time: as many trips to memory as reading the item from a list, and a few hundred instructions.  What it saves is a kernel in front; what it
// costs are those instructions, item by item (where they cost more, a kernel makes the list after all, list_items_kernel), so it is a level
// search of one pass where lanes and sequences are few, and prefixes come from counts of set bits.  Whole call, against the list of a
// single workgroup: 2 759 tokens, 16 heads on 2 27.0 -> 22.9 us; 16 384 tokens in 15 sequences, 16 heads on 2 152.5 -> 150.3.
// And tiles that outlast the rest are cut into parts as a plan cuts them (split_long_items; the same parts, as long as the records of
// partial results suffice), which a list of whole tiles did not: 63 259 tokens, 1 head 167 -> 112 us; 51 606, 2 heads on 1 146.3 -> 143.3.
// Only where the longest tile outlasts the rest by more than the hand-over costs.  A workgroup whose neighbour on the compute unit has run out
// of work goes nearly twice as fast, so a longest tile that is alone there costs time from about two even shares on, and beyond that must be worth
// the hand-over's steps; without a mask all tiles of the longest sequence are equally long, and where they are more than the compute
// units two of them share one.  Whole call, whole -> cut: 6 208 tokens in four sequences, 16 heads on 4 (a share of 34 steps, the longest
// 59) 80 -> 88 us; 10 994 in 171, 12 heads, D = 64 (48, 86) 83 -> 91; a share of 64 to 96 steps and 2 to 2.3 of it 0.94 of the time, up to 48 steps 1.04 to 1.09;
// unmasked 38 098, 2 heads, D = 64 (233, 338, on 338 tiles) 319 -> 270; 6 773, 6 heads on 3 (20, 58, on 174 tiles) 55 -> 70.  Of 618 batches whose longest
// tile lasts a share or more, cut by this line, eight take over 2 % more than whole (cut from 1.4 shares on, 186).
template <int CHUNKS>
struct SearchBatch {
    static constexpr int kWhole = 1 << 24;  // a part length that no tile reaches
    int total;   // places
    int maxnt;   // query tiles of the longest sequence
    int target;  // steps of a part

    struct Lens {
        int lo, len, nt;
        __device__ __forceinline__ int steps() const { return (len + kFwdBk - 1) / kFwdBk; }  // key tiles of the last query tile
    };
    __device__ __forceinline__ static Lens lens(KernArgs &a, int b)
    {
        Lens l;
        l.lo = b < a.B ? a.cu[b] : 0;
        l.len = b < a.B ? a.cu[b + 1] - l.lo : 0;
        l.nt = (l.len + kFwdBq - 1) / kFwdBq;
        return l;
    }
    // parts of a tile of c steps (part_count): n of them from least(n) steps on
    __device__ __forceinline__ int least(int n) const { return max((n - 1) * target + 1, n * kMinPartSteps); }
    __device__ __forceinline__ int parts(int c) const
    {
        int k = 1;
#pragma unroll
        for (int n = 2; n <= kMaxParts; n++) k += c >= least(n);
        return k;
    }
    // causal: first level whose tiles have n parts; parts of the tiles below level n together (a sequence's last tile apart)
    __device__ __forceinline__ int first_level(int n) const { return (least(n) + 1) / 2 - 1; }
    __device__ __forceinline__ int below(int level) const
    {
        int s = level;
#pragma unroll
        for (int n = 2; n <= kMaxParts; n++) s += max(0, level - first_level(n));
        return s;
    }
    // all parts of a sequence
    __device__ __forceinline__ int all_parts(const Lens &l, int causal) const
    {
        const int k = parts(l.steps());
        return l.nt <= 0 ? 0 : causal ? below(l.nt - 1) + k : l.nt * k;
    }
    // ... at `level` and above (`all`: all_parts)
    __device__ __forceinline__ static int from_level(const Lens &l, int all, int level, int below_level, int causal)
    {
        return level < l.nt ? all - (causal ? below_level : 0) : 0;
    }

    __device__ __forceinline__ SearchBatch(KernArgs &args, int lane)
    {
        KernArgs &a = fresh(args);
        static_assert(kFwdBq == 2 * kFwdBk, "a query tile is two key tiles");
        const int causal = a.causal, heads = a.Hq;
        const int first = a.cu[0], last = a.cu[a.B];
        Lens l[CHUNKS];
        int cost = 0, longest = 0;
        bool bad = __builtin_amdgcn_readfirstlane(first) != 0;
#pragma unroll
        for (int c = 0; c < CHUNKS; c++) {
            l[c] = Lens{0, 0, 0};
            if (c * 64 >= a.B) continue;
            l[c] = lens(a, c * 64 + lane);
            bad = bad || __builtin_amdgcn_ballot_w64(l[c].lo < 0 || l[c].len < 0 || l[c].len > a.T - l[c].lo) != 0;
            cost += causal ? l[c].nt * (l[c].nt - 1) + l[c].steps() : l[c].nt * l[c].steps();
            longest = max(longest, l[c].nt);
        }
        total = maxnt = 0;
        target = kWhole;
        if (bad) return;
        maxnt = lanes_max(longest);
        // (no parts where a call on tensors of the batch's own size would be one of few items, which has none: the room in the tensors
        // changes no bits)
        const int share = (int)((int64_t)lanes_sum(cost) * heads / (2 * a.num_cu)), steps = 2 * maxnt;
        int longs = 0;  // without a mask: tiles of three quarters of the longest's steps or more
        if (!causal) {
#pragma unroll
            for (int c = 0; c < CHUNKS; c++) longs += 4 * l[c].nt >= 3 * maxnt ? l[c].nt : 0;
            longs = lanes_sum(longs) * heads;
        }
        const bool outlasts = causal ? 4 * steps > 7 * share + 80 : longs <= a.num_cu ? steps > 2 * share + 20 : 3 * steps > 4 * share + 42;
        if (((__builtin_amdgcn_readfirstlane(last) + kFwdBq - 1) / kFwdBq + a.B) * (int64_t)heads > 2 * a.num_cu && outlasts) {
            target = max(min(share * 3 / 4, max((int)((int64_t)share * 35 / 100), (int)kLongPartSteps)), kMinPartSteps);
        }
        // (every cut tile stands at a level from first_level(2) on: a record for each place down to there.  Too few: longer parts for all tiles,
        // which keeps what a place holds a matter of its tile alone)
        for (;; target *= 2) {
            const int cut_level = first_level(2), cut_below = below(cut_level);
            int all = 0, cut = 0;
#pragma unroll
            for (int c = 0; c < CHUNKS; c++) {
                if (c * 64 >= a.B) continue;
                const int n = all_parts(l[c], causal);
                all += n;
                cut += from_level(l[c], n, cut_level, cut_below, causal);
            }
            if (cut_level >= maxnt || lanes_sum(cut) * heads <= kStaticRecords) {
                total = lanes_sum(all) * heads;
                return;
            }
        }
    }

    __device__ __forceinline__ flexsp_item item(KernArgs &a, int place, int lane) const
    {
        SearchBatch here = *this;  // (what follows from the part length is not worth keeping from item to item)
        asm volatile("" : "+s"(here.target), "+v"(lane));
        return here.find(a, place, lane);
    }
    __device__ __forceinline__ flexsp_item find(KernArgs &a, int place, int lane) const
    {
        const int heads = a.Hq, group = heads / kMaxQueues;
        int pos, h;
        if (heads % kMaxQueues) {
            pos = place / heads;
            h = place - pos * heads;
        } else {  // neighbouring heads share a queue (see nth_head in flexsp_host.hip)
            const int l = place / kMaxQueues;
            pos = l / group;
            h = place % kMaxQueues * group + l - pos * group;
        }
        return head_of(tile(a, pos, lane), h);
    }
    // ... and the other way round: the queue of position pos of head h, and the place there
    __device__ __forceinline__ static int2 queue_place(int heads, int pos, int h)
    {
        const int group = heads / kMaxQueues, place = pos * heads + h;
        return heads % kMaxQueues ? int2{place % kMaxQueues, place / kMaxQueues} : int2{h / group, pos * group + h % group};
    }
    __device__ __forceinline__ static flexsp_item head_of(flexsp_item it, int h)
    {
        it.head = h;
        if (it.slot >= 0) it.slot += h * (it.parts & 0xffff);
        return it;
    }
    // What stands at a position, the same for every head: a tile of the first, or a part of one
    __device__ __forceinline__ flexsp_item tile(KernArgs &a, int pos, int lane) const
    {
        const int causal = a.causal, heads = a.Hq;
        Lens l[CHUNKS];
        int all[CHUNKS];
#pragma unroll
        for (int c = 0; c < CHUNKS; c++) {
            l[c] = Lens{0, 0, 0};
            all[c] = 0;
            if (c * 64 < a.B) {
                l[c] = lens(a, c * 64 + lane);
                all[c] = all_parts(l[c], causal);
            }
        }
        int level = 0, before = 0;  // places from `level` on: more than pos; above it, `before` of them: not
        if (maxnt <= 64 && a.B <= 32) {  // a lane to a level
            const int below_mine = below(lane);
            int n = 0;
            for (int b = 0; b < a.B; b++) {
                const int nt = __builtin_amdgcn_readlane(l[0].nt, b), n_all = __builtin_amdgcn_readlane(all[0], b);
                n += lane < nt ? n_all - (causal ? below_mine : 0) : 0;
            }
            level = 63 - __builtin_clzll(__builtin_amdgcn_ballot_w64(n > pos));
            before = level == 63 ? 0 : __builtin_amdgcn_readlane(n, level + 1);
        } else {
            for (int above = maxnt; above - level > 1;) {
                const int m = (level + above) / 2, below_m = below(m);
                int n = 0;
#pragma unroll
                for (int c = 0; c < CHUNKS; c++)
                    if (c * 64 < a.B) n += from_level(l[c], all[c], m, below_m, causal);
                n = lanes_sum(n);
                if (n > pos) {
                    level = m;
                } else {
                    above = m;
                    before = n;
                }
            }
        }
        // Which sequence of this level, which of its parts there.  The last tile of a sequence may be a step shorter than the others of its
        // level, and have other parts: two kinds of sequences.
        const int k_whole = parts(2 * level + 2), k_less = parts(2 * level + 1), tiles = causal ? 1 : level + 1;
        flexsp_item it = {};
        int rem = pos - before;
#pragma unroll
        for (int c = 0; c < CHUNKS; c++) {
            if (c * 64 >= a.B) continue;
            const bool here = causal ? level < l[c].nt : level == l[c].nt - 1;
            const bool less = here && level == l[c].nt - 1 && (l[c].steps() & 1);
            const uint64_t m_less = __builtin_amdgcn_ballot_w64(less), m_whole = __builtin_amdgcn_ballot_w64(here) & ~m_less;
            const int n = here ? (less ? k_less : k_whole) * tiles : 0;
            const int from = (__builtin_amdgcn_mbcnt_hi(m_whole >> 32, __builtin_amdgcn_mbcnt_lo((uint32_t)m_whole, 0)) * k_whole +
                              __builtin_amdgcn_mbcnt_hi(m_less >> 32, __builtin_amdgcn_mbcnt_lo((uint32_t)m_less, 0)) * k_less) * tiles;
            const uint64_t owner = __builtin_amdgcn_ballot_w64(rem >= from && rem < from + n);
            if (owner) {
                const int w = __builtin_ctzll(owner);
                int part = rem - __builtin_amdgcn_readlane(from, w);
                const int np = m_less >> w & 1 ? k_less : k_whole;
                it.seq_start = __builtin_amdgcn_readlane(l[c].lo, w);
                it.seq_len = __builtin_amdgcn_readlane(l[c].len, w);
                it.tile = level;
                if (!causal) {
                    it.tile = part / np;
                    part -= it.tile * np;
                }
                const int steps = ((causal ? min(it.seq_len, (it.tile + 1) * kFwdBq) : it.seq_len) + kFwdBk - 1) / kFwdBk;
                it.step_begin = np > 1 ? part * steps / np : 0;
                it.step_end = np > 1 ? (part + 1) * steps / np : steps;
                it.slot = np > 1 ? (pos - part) * heads : -1;
                it.parts = part << 16 | np;
                rem = -1;
            }
            if (rem >= 0) rem -= (__builtin_popcountll(m_whole) * k_whole + __builtin_popcountll(m_less) * k_less) * tiles;
        }
        return it;
    }
};

}  // namespace
}  // namespace flexsp
