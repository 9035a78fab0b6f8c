// Forward of packed causal attention (paper Sec. 2.1.2, Eq. 3, evaluated per sequence of
// the packed stream, Sec. 2.2.2) for gfx950.
//
// One work item = 128 query rows of one (sequence, head).  A workgroup of 4 wavefronts
// takes items from the longest-first queues until they are empty.  Each wavefront owns 32
// query rows and keeps their Q in registers.  Key/value tiles of 64 rows go straight from
// global memory into swizzled LDS tiles (no staging registers), double-buffered, one barrier
// per tile.
//
// The score block is computed TRANSPOSED, S^T = K Q^T, so that in the 32x32 accumulator a
// lane holds one query (its column) and 16 keys: the row-wise softmax is a reduction over a
// lane's own registers plus one exchange with the lane 32 away, and the exponentiated block,
// rounded to bf16, is directly the B operand of O^T += V^T P^T.  V^T fragments come from
// the row-major V tile through the LDS transpose read.  The running output is rescaled only
// when some row's maximum actually grew.
//
// A wavefront walks the keys in blocks of 32 (two per tile) as a software pipeline: iteration
// c issues the matrix instructions of S(c+1) and of O += P(c-1) V(c-1) and, between them, the
// softmax arithmetic of block c, so that the matrix pipe and the vector pipe of the SIMD work
// at the same time inside one wavefront (the file is compiled with the compiler's
// pre-allocation schedulers off: the order written here is the order executed).  The K tiles
// therefore run one tile ahead of the V tiles: between the barriers of tile t and t+1 the
// wavefronts read K tile t+1 and V tile t while K tile t+2 and V tile t+1 are in flight.
#pragma once

#include <type_traits>

#include "attn_common.h"

namespace flexsp {
namespace {

template <int V>
using ic = std::integral_constant<int, V>;

// The n-th item of a batch, items counted by query tile of the packed sequences and then by head, as wave-uniform values; every
// wavefront looks for itself, 64 sequences at a time.  False if there are fewer items or the lengths are not 0 = cu[0] <=
// cu[1] <= ... <= cu[B] <= T.
__device__ __forceinline__ bool find_item(const int32_t *cu, int B, int T, int heads, int causal, int n, int lane, flexsp_item &it)
{
    const int pair = n / heads;
    int before = 0, start = 0, len = 0, tile = -1;
    bool bad = cu[0] != 0;
    for (int b0 = 0; b0 < B; b0 += 64) {
        const int b = b0 + lane;
        const int lo = b < B ? cu[b] : 0, hi = b < B ? cu[b + 1] : 0;
        const bool wrong = lo < 0 || hi < lo || hi > T;
        bad = bad || wrong;
        const int nt = wrong ? 0 : (hi - lo + kFwdBq - 1) / kFwdBq;
        int upto = nt;  // tiles of this and the earlier lanes
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            const int x = __shfl_up(upto, d);
            if (lane >= d) upto += x;
        }
        const uint64_t mine = __builtin_amdgcn_ballot_w64(pair >= before + upto - nt && pair < before + upto);
        if (mine) {
            const int l = __builtin_ctzll(mine);
            start = __builtin_amdgcn_readlane(lo, l);
            len = __builtin_amdgcn_readlane(hi, l) - start;
            tile = pair - before - __builtin_amdgcn_readlane(upto - nt, l);
        }
        before += __builtin_amdgcn_readlane(upto, 63);
    }
    if (tile < 0 || __builtin_amdgcn_ballot_w64(bad) != 0) return false;
    it.seq_start = start;
    it.seq_len = len;
    it.tile = tile;
    it.head = n - pair * heads;
    it.step_begin = 0;
    it.step_end = ((causal ? min(len, (tile + 1) * kFwdBq) : len) + kFwdBk - 1) / kFwdBk;
    it.slot = -1;
    it.parts = 1;
    return true;
}

// The lengths of a batch of at most 64 sequences, a lane each, where they also say whether the batch runs in halves: find_item for
// tiles of either size from one look at them, one chain of exchanges.
template <int D>
struct ShortBatch {
    int lo, hi;
    uint32_t n, upto;  // tiles of kHalfBq rows | tiles of kFwdBq rows << 16: this lane's, and with those of the earlier ones
    bool bad, halves;

    __device__ __forceinline__ ShortBatch(KernArgs &a, int lane)
    {
        const int32_t *cu = a.cu;
        const int B = a.B, heads = a.Hq;
        lo = lane < B ? cu[lane] : 0, hi = lane < B ? cu[lane + 1] : 0;
        const int first = cu[0], total = cu[B];
        const bool wrong = lo < 0 || hi < lo || hi > a.T;
        bad = first != 0 || __builtin_amdgcn_ballot_w64(wrong) != 0;
        const int len = wrong ? 0 : hi - lo, h = (len + kHalfBq - 1) / kHalfBq;
        n = upto = h | (len + kFwdBq - 1) / kFwdBq << 16;
        int steps = a.causal ? h * (h + 1) / 2 : h * h, longest = h;
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            const uint32_t x = __shfl_up(upto, d);
            if (lane >= d) upto += x;
            steps += __shfl_xor(steps, d);
            longest = max(longest, __shfl_xor(longest, d));
        }
        const int tiles = __builtin_amdgcn_readlane(upto, 63) & 0xffff;
        steps = __builtin_amdgcn_readfirstlane(steps);
        longest = __builtin_amdgcn_readfirstlane(longest);
        halves = fwd_halves(D, {total, B, (int64_t)tiles * heads, (int64_t)steps * heads, longest}, a.num_cu);
    }
    __device__ __forceinline__ bool item(KernArgs &a, int n_th, flexsp_item &it) const
    {
        const int pair = n_th / a.Hq, shift = halves ? 0 : 16, rows = halves ? kHalfBq : kFwdBq;
        const int end = upto >> shift & 0xffff, mine = n >> shift & 0xffff;
        const uint64_t owner = __builtin_amdgcn_ballot_w64(pair >= end - mine && pair < end);
        if (bad || !owner) return false;
        const int l = __builtin_ctzll(owner);
        it.seq_start = __builtin_amdgcn_readlane(lo, l);
        it.seq_len = __builtin_amdgcn_readlane(hi, l) - it.seq_start;
        it.tile = pair - __builtin_amdgcn_readlane(end - mine, l);
        it.head = n_th - pair * a.Hq;
        it.step_begin = 0;
        it.step_end = ((a.causal ? min(it.seq_len, (it.tile + 1) * rows) : it.seq_len) + kFwdBk - 1) / kFwdBk;
        it.slot = -1;
        it.parts = 1;
        return true;
    }
};

// SHARD = true is the variant for one shard of the keys (context parallelism): a work item then
// names separate query and key ranges and an offset `shift` between their positions, key j is
// visible to query row i iff j <= i + shift (when causal), rows may see no key at all (O = 0,
// LSE = -inf), and up to three 32-key blocks of a wavefront need masking (the diagonal crosses two
// when shift is not a multiple of 32, plus the ragged end of the shard).
//
// FIND = true is the variant without a list of items: workgroup w finds the w-th (query tile, head) of the batch in the
// lengths and leaves when it is done.
//
// BATCH (attn_fwd_search.hip) is what finds an item in the lengths where there is no list either, but more items than workgroups: they are
// dealt by their places in the list that there would be.
//
// HALVES = 2 is the variant for launches that leave compute units without work: a workgroup is 64 query rows, half an item, and two
// wavefronts to each block of 32 rows: wavefronts 0 and 1 walk the first half of the key tiles, 2 and 3 the second, each pair with
// tiles of its own, and hand over through LDS.  Such a launch lasts as long as its longest item's chain of steps, and a step lasts
// as long as one wavefront's matrix instructions; a hand-over through memory costs what the shorter chain saves.
//
// BUFS = 1 has one buffer for K and one for V instead of two and waits for every tile: halves with the LDS of whole items, for launches
// sized for those whose batch turns out to be one for halves.
template <int D, int HALVES, int BUFS>
constexpr int fwd_lds()  // bytes of LDS of the pass: [K buffers | V buffers], each half of the wavefronts its own
{
    return HALVES * 2 * BUFS * kFwdBk * LdsTile<D>::ROWB;
}
template <int HALVES>
constexpr int fwd_stats()  // floats of LDS for the second half's row maxima and sums
{
    return HALVES == 2 ? kThreads : 2;
}
struct NoBatch {};
template <int D, bool SHARD, bool FIND, int HALVES, int BUFS = 2, class BATCH = NoBatch>
__device__ __forceinline__ void fwd_pass(KernArgs &args, const flexsp_item &found, char *const smem, float *const stats, int &deal_word, int &split_word,
                                         const BATCH &batch = BATCH())
{
    static_assert(HALVES == 1 || !SHARD, "no list of a shard's launch asks for it");
    static_assert(BUFS == 2 || HALVES == 2, "whole items have two buffers");
    typedef LdsTile<D> L;
    constexpr int KS = D / 16;                  // k steps of the score product
    constexpr int DB = D / 32;                  // 32-wide blocks of the head dim
    constexpr int TILE = kFwdBk * L::ROWB;      // bytes of one 64-row tile
    constexpr int NT = kThreads / HALVES;       // threads that share a tile
    constexpr int BQ = kFwdBq / HALVES;         // query rows of the workgroup
    constexpr int NCP = 2 * kFwdBk * L::CH / NT;  // copy instructions per wavefront for a K and a V tile
    constexpr int NSLOT = KS + 2 * DB;          // matrix instructions of one pipeline iteration
    static_assert(NSLOT * HALVES == 2 * NCP, "one copy instruction per two matrix instructions, or per one");
    constexpr int REGION = 2 * BUFS * TILE;     // LDS of a half of the wavefronts
    static_assert(fwd_lds<D, HALVES, BUFS>() == HALVES * REGION && fwd_stats<HALVES>() >= HALVES * NT * (HALVES - 1), "LDS of the pass");

    const int tid = thread_id();
    const int lane0 = tid & 63;
    const int wave4 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = HALVES == 2 ? wave4 & 1 : wave4, half = HALVES == 2 ? wave4 >> 1 : 0;
    char *const mine = smem + half * REGION;  // for copies and stores; reads of tiles have the half in their lane offsets:
    LaneOffsets<D> lo;
    lo.init(lane0);
    if constexpr (HALVES == 2) {
#pragma unroll
        for (int ks = 0; ks < KS; ks++) lo.nat[ks] += half * REGION;
#pragma unroll
        for (int db = 0; db < DB; db++) lo.tr[db][0] += half * REGION, lo.tr[db][1] += half * REGION;
    }
    constexpr bool SEARCH = !std::is_same<BATCH, NoBatch>::value;
    Dealer<!SEARCH> deal;

    int item;
    if constexpr (FIND) {
        deal.direct = true;
        item = 0;
    } else if constexpr (HALVES == 2) {
        deal.direct = true;
        item = workgroup_id();
    } else {
        if constexpr (SEARCH) deal.total = batch.total;
        item = deal.first(args.pq, args.grid, 0, &deal_word, wave, lane0);
    }
    for (; item >= 0; item = deal.advance()) {
        KernArgs &a = fresh(args);
        // s: query rows of the sequence; sk: its keys; tok0 / ktok0: their first rows in q / k, v
        int s, sk, shift, h, q0;
        int64_t tok0, ktok0;
        int part = 0, nparts = 1, slot = -1, t_lo = 0, t_hi = 0;  // (see flexsp_item): the item walks key tiles t_lo .. t_hi-1
        if constexpr (SHARD) {
            const flexsp_shard_item it = load_shard_item((const flexsp_shard_item *)a.pq.items, item);
            s = it.q_len; sk = it.k_len; shift = it.shift; h = it.head_parts & 0xffff; q0 = it.tile * kFwdBq;
            tok0 = it.q_start; ktok0 = it.k_start;
            // (a part of a cut tile comes with its own key range and shift: nothing else differs)
            part = (it.head_parts >> 16) & 0xff; nparts = it.head_parts >> 24; slot = it.slot;
        } else {
            flexsp_item it;
            if constexpr (FIND) it = uniform_item(found); else if constexpr (SEARCH) it = batch.item(a, item, lane0); else it = load_item(a.pq.items, item);
            s = it.seq_len; sk = s; shift = 0; h = it.head; q0 = it.tile * BQ;
            tok0 = it.seq_start; ktok0 = tok0;
            part = it.parts >> 16; nparts = it.parts & 0xffff; slot = it.slot;
            t_lo = it.step_begin; t_hi = it.step_end;
        }
        // opaque per-item copy of the lane id: per-lane address arithmetic of an item stays inside
        // the item instead of being hoisted out of this loop into long-lived registers
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        lane &= 63;  // (its range is known again: divisions by the pieces of a row are shifts)
        const int r = lane & 31, hl = lane >> 5;
        const int g = h / a.G;
        // keys this item needs
        int kv_end = SHARD ? (a.causal ? max(0, min(sk, q0 + BQ + shift)) : sk)
                           : (a.causal ? min(s, q0 + BQ) : s);
        // this half's key tiles; windows, and with them barriers, of the first half (the second has no more)
        int windows = 0;
        if constexpr (HALVES == 2) {
            const int n = (kv_end + kFwdBk - 1) / kFwdBk, first = n >= kSplitSteps ? (n + 1) / 2 : n;
            windows = first;
            t_lo = half ? first : 0;
            t_hi = half ? n : first;
        }
        // The item walks key tiles t_lo .. t_hi-1 (all of them unless the tile was cut).  From here on keys are counted
        // from the part's first one (koff keys are skipped: a multiple of the tile size, so blocks
        // stay aligned and still at most one block per wavefront needs masking); a wavefront whose
        // rows see none of the part's keys (the part after the diagonal of the tile's upper rows) ends
        // with maximum -inf and sum 0, which the merge below weighs with zero.
        int koff = 0;
        if constexpr (!SHARD) {
            koff = t_lo * kFwdBk;
            kv_end = min(kv_end, t_hi * kFwdBk) - koff;
            sk = s - koff;
            ktok0 += koff;
        }
        if constexpr (SHARD) {
            if (kv_end <= 0) {
                // no row of this item sees a key of the shard: O = 0, LSE = -inf (the neutral element
                // of the merge); deal.advance() holds the barrier every item ends with
                if (a.dq) {
                    // folding into a running result: it stays as it is; only its bf16 copy, if asked for, is written
                    if (a.out_o) {
                        for (int idx = tid; idx < kFwdBq * L::CH; idx += kThreads) {
                            const int row = q0 + idx / L::CH;
                            if (row >= s) continue;
                            const bool live = a.delta_out[(int64_t)h * a.T + tok0 + row] > -INFINITY;
                            const float *src = (const float *)a.dq + (tok0 + row) * a.dq_st + (int64_t)h * a.dq_sh + (idx % L::CH) * 8;
                            const f32x4 x0 = *(const f32x4 *)src, x1 = *(const f32x4 *)(src + 4);
                            u32x4 y = {pack_bf16x2(x0[0], x0[1]), pack_bf16x2(x0[2], x0[3]), pack_bf16x2(x1[0], x1[1]),
                                       pack_bf16x2(x1[2], x1[3])};
                            if (!live) y = u32x4{0, 0, 0, 0};
                            *(u32x4 *)(a.out_o + (tok0 + row) * a.o_st + (int64_t)h * a.o_sh + (idx % L::CH) * 8) = y;
                        }
                    }
                    deal.prefetch();
                    continue;
                }
                for (int idx = tid; idx < kFwdBq * L::CH; idx += kThreads) {
                    const int row = q0 + idx / L::CH;
                    if (row < s)
                        *(u32x4 *)(a.out_o + (tok0 + row) * a.o_st + (int64_t)h * a.o_sh + (idx % L::CH) * 8) =
                            u32x4{0, 0, 0, 0};
                }
                if (tid < kFwdBq && q0 + tid < s) a.lse_out[(int64_t)h * a.T + tok0 + q0 + tid] = -INFINITY;
                deal.prefetch();
                continue;
            }
        }
        const int ntiles = (kv_end + kFwdBk - 1) / kFwdBk;
        const uint16_t *kbase = a.k + ktok0 * a.k_st + (int64_t)g * a.k_sh;
        const uint16_t *vbase = a.v + ktok0 * a.v_st + (int64_t)g * a.v_sh;

        constexpr int CP_ = TileCopy<D, NT>::P;
        uint32_t goffk[CP_], goffv[CP_];
#pragma unroll
        for (int n = 0; n < CP_; n++) goffk[n] = tile_goff<D, NT>(a.k_st, wave, lane, n), goffv[n] = tile_goff<D, NT>(a.v_st, wave, lane, n);
        auto copy_one = [&](char *dst, const uint16_t *src, int32_t st, const uint32_t (&goff)[CP_], int n) {
            load_tile_async_fast_one<D, NT>(dst, src, st, goff[n % CP_], wave, n);
        };
        // whole-tile copies (all of this wavefront's copy instructions back to back)
        auto prefetch_k = [&](int t, int buf) {
            char *dst = mine + buf * TILE;
            if ((t + 1) * kFwdBk <= sk)  // whole tile inside the sequence
#pragma unroll
                for (int n = 0; n < NCP / 2; n++) copy_one(dst, kbase + (int64_t)t * kFwdBk * a.k_st, a.k_st, goffk, n);
            else
                load_tile_async<D, kFwdBk, NT>(dst, kbase, a.k_st, t * kFwdBk, sk - 1, wave, lane);
        };
        auto prefetch_v = [&](int t, int buf) {
            char *dst = mine + (BUFS + buf) * TILE;
            if ((t + 1) * kFwdBk <= sk)
#pragma unroll
                for (int n = 0; n < NCP / 2; n++) copy_one(dst, vbase + (int64_t)t * kFwdBk * a.v_st, a.v_st, goffv, n);
            else
                load_tile_async<D, kFwdBk, NT>(dst, vbase, a.v_st, t * kFwdBk, sk - 1, wave, lane);
        };
        if (HALVES == 1 || ntiles > 0) prefetch_k(0, 0);

        // ---- Q fragments (B operand: column = query row, k = head dim), kept in registers: the rows
        // are requested here and become fragments just before the barrier below
        const int qrow = q0 + wave * 32 + r;  // row inside the sequence
        const int wq_lo = q0 + wave * 32;     // smallest query row of this wavefront
        RowBlock<D> qrows;
        qrows.load(a.q + tok0 * a.q_st + (int64_t)h * a.q_sh, a.q_st, wq_lo, s - 1, lane);
        bf16x8 qf[KS];
        // last 32-key block this wavefront has to look at (-1: none, its rows lie past the sequence)
        int cmax, cmask, lim;
        if constexpr (SHARD) {
            // (>> of a negative number rounds down: a diagonal left of the shard gives a negative block)
            cmax = wq_lo >= s ? -1 : max(-1, a.causal ? min((kv_end - 1) >> 5, (wq_lo + 31 + shift) >> 5) : (kv_end - 1) >> 5);
            cmask = a.causal ? min((wq_lo + shift) >> 5, (sk - 1) >> 5) : ((sk - 1) >> 5);  // FIRST block that needs masking
            lim = a.causal ? min(qrow + shift, sk - 1) : sk - 1;
        } else {
            // (wq_lo - koff is negative for rows that lie before the part's keys: >> rounds down, no block)
            cmax = wq_lo >= s ? -1 : (a.causal ? min((kv_end - 1) >> 5, (wq_lo - koff) >> 5) : (kv_end - 1) >> 5);
            cmask = a.causal ? ((wq_lo - koff) >> 5) : ((sk - 1) >> 5);  // the block that needs masking
            lim = a.causal ? qrow - koff : sk - 1;                        // largest visible key of this lane's row
        }

        f32x16 oacc[DB];
#pragma unroll
        for (int db = 0; db < DB; db++)
#pragma unroll
            for (int i = 0; i < 16; i++) oacc[db][i] = 0.f;
        // (SHARD: a finite floor instead of -inf, because a row may have every key of a block masked:
        // its scores are -inf, and -inf minus a reference of -inf would not be a number)
        float m_run = SHARD ? -1e30f : -INFINITY, l_run = 0.f;
        float psum_max = 0.f;  // largest row sum of a block taken without its maximum (see iter_fast)
        f32x16 sacc[2];     // S of block c in sacc[c & 1]
        uint32_t pk[2][8];  // P of block c (bf16 pairs) in pk[c & 1]
        // Blocks are computed under conditions, so to the compiler the arrays' contents pass from item to item, 48 registers
        // of them, which SHARD stored and loaded around every item: 128 spilled vector registers with D = 128.  An item
        // that defines them itself, as anything, left 29 of them (none by now).  Shard forwards of a 64K-token batch over four devices, plain and folding,
        // 346 -> 262 and 498 -> 310 us; of 93-token sequences over eight, 3 655 -> 1 605 and 5 050 -> 2 111 us.
#pragma unroll
        for (int j = 0; j < 2; j++) {
            asm volatile("" : "=v"(sacc[j]));
#pragma unroll
            for (int i = 0; i < 8; i++) asm volatile("" : "=v"(pk[j][i]));
        }

        // ---------------- the three stages of a block, one after the other (pipeline ends) -----
        // S(c) = K(c) Q^T; `sK` points at the block's first row inside its K tile
        auto scores = [&](f32x16 &sa, const char *sK) {
            constexpr int AH = 4;
            bf16x8 kf[KS];
#pragma unroll
            for (int i = 0; i < 16; i++) sa[i] = 0.f;
#pragma unroll
            for (int j = 0; j < AH && j < KS; j++) kf[j] = lds_nat(sK, lo.nat[j]);
#pragma unroll
            for (int j = 0; j < KS; j++) {
                if (j + AH < KS) kf[j + AH] = lds_nat(sK, lo.nat[j + AH]);
                sa = mfma32(kf[j], qf[j], sa);
            }
        };
        // O^T += V(c)^T P(c)^T
        auto pv = [&](const uint32_t (&p)[8], const char *sV) {
            constexpr int AH = 4, N = 2 * DB;
            bf16x8 vf[N];
            auto vread = [&](int j) {
                const int rowoff = (j / DB) * 16 * L::ROWB;
                return lds_tr(sV, rowoff + lo.tr[j % DB][0], rowoff + lo.tr[j % DB][1]);
            };
#pragma unroll
            for (int j = 0; j < AH && j < N; j++) vf[j] = vread(j);
#pragma unroll
            for (int j = 0; j < N; j++) {
                if (j + AH < N) vf[j + AH] = vread(j + AH);
                const int st = j / DB;
                Frag8 pf;
                pf.u = u32x4{p[4 * st], p[4 * st + 1], p[4 * st + 2], p[4 * st + 3]};
                oacc[j % DB] = mfma32(vf[j], pf.v, oacc[j % DB]);
            }
        };
        // Online-softmax bookkeeping shared by both forms of an iteration.
        //   row maximum of a block: own 16 keys, then the other half-wave's
        auto block_max = [&](const f32x16 &sa) {
            float mx = fmaxf(sa[0], sa[1]);
#pragma unroll
            for (int i = 2; i < 16; i += 2) mx = fmaxf(mx, fmaxf(sa[i], sa[i + 1]));
            return halves_max(mx);
        };
        //   the reference value subtracted from a block's scores: the running one, which only moves
        //   when some row's maximum exceeds it by more than 8 in the exponent's units (P then stays
        //   below 2^8: exact in bf16 and fp32 alike, and the final O / l and LSE do not depend on
        //   the reference).  Without the slack the first blocks of every item, where the maxima still
        //   grow a little with each block, would rescale O (64 multiplications) almost every time.
        const float slack = 8.0f / a.scale_l2;
        auto reference = [&](float mx) {
            const bool move = __builtin_amdgcn_ballot_w64(mx > m_run + slack) != 0;
            return move ? fmaxf(m_run, mx) : m_run;
        };
        //   after the iteration's O += P V: rescale if the reference moved, fold in the row sums
        auto finish_block = [&](float m_new, float psum) {
            if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
                const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * a.scale_l2);
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < DB; db++)
#pragma unroll
                    for (int i = 0; i < 16; i++) oacc[db][i] *= alpha;
                m_run = m_new;
            }
            l_run += psum;  // fp32: the log-sum-exp feeds the backward recomputation
        };

        // ---------------- iteration c, general form: any subset of the three stages ------------
        // S(c+1), softmax(c), O += P(c-1) V(c-1), done one after the other.  Used where the pipeline
        // fills and drains and for the masked block.  sK / sV: first row of block c+1 / c-1.
        auto iter_slow = [&](auto cpc, int c, const char *sK, const char *sV) {
            constexpr int CP = decltype(cpc)::value;  // c & 1
            if (c + 1 <= cmax) scores(sacc[CP ^ 1], sK);
            float m_new = m_run, psum = 0.f;
            if (c <= cmax) {
                f32x16 &sa = sacc[CP];
                if (SHARD ? c >= cmask : c == cmask) {
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        const int kv = c * 32 + 8 * (i >> 2) + 4 * hl + (i & 3);
                        if (kv > lim) sa[i] = -INFINITY;
                    }
                }
                m_new = reference(block_max(sa));
                const float moff = m_new * a.scale_l2;
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sa[i], a.scale_l2, -moff));
                    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sa[i + 1], a.scale_l2, -moff));
                    psum += p0 + p1;
                    pk[CP][i >> 1] = pack_bf16x2(p0, p1);
                }
            }
            if (c >= 1 && c - 1 <= cmax) pv(pk[CP ^ 1], sV);
            if (c <= cmax) finish_block(m_new, psum);
        };

        // ---------------- iteration c, pipelined form: all three stages, interleaved -----------
        // Slot j issues matrix instruction j (first the KS of S(c+1), then the 2*DB of O += P V),
        // the LDS read of the operand AH slots ahead, every second slot one copy instruction of the
        // tiles in flight (PF; K tile t+2 and V tile t+1), and a share of the softmax arithmetic of
        // block c: the row maximum in slots 0 and 1, the 16 exponentials over the remaining slots.
        // One basic block on purpose: a branch inside it would let the optimiser sink the softmax
        // arithmetic below the matrix instructions.
        auto iter_fast = [&](auto cpc, auto kbc, auto vbc, auto pfc, int t) {
            constexpr int CP = decltype(cpc)::value;  // c & 1; blocks c+1 and c-1 start at row 0 (CP = 1) or 32 of their tile
            constexpr int KB = decltype(kbc)::value, VB = decltype(vbc)::value;
            constexpr bool PF = decltype(pfc)::value != 0;
            constexpr int AH = 4;
            const char *sK = smem + KB * TILE + (CP ? 0 : 32 * L::ROWB);
            const char *sV = smem + (BUFS + VB) * TILE + (CP ? 0 : 32 * L::ROWB);
            f32x16 &sn = sacc[CP ^ 1];
            const f32x16 &sc = sacc[CP];
            const uint32_t(&pp)[8] = pk[CP ^ 1];
            bf16x8 fr[NSLOT];
            auto rd = [&](int j) {
                if (j < KS) return lds_nat(sK, lo.nat[j < KS ? j : 0]);
                const int rowoff = ((j - KS) / DB) * 16 * L::ROWB;
                return lds_tr(sV, rowoff + lo.tr[(j - KS) % DB][0], rowoff + lo.tr[(j - KS) % DB][1]);
            };
#pragma unroll
            for (int j = 0; j < AH; j++) fr[j] = rd(j);
#pragma unroll
            for (int i = 0; i < 16; i++) sn[i] = 0.f;
            // The block's scores are taken against the running reference as it stands, without looking
            // at their maximum first: bf16 and fp32 share their exponent range, so P may grow far
            // beyond 1 before anything is lost (O and the row sums are accumulated in fp32 and divided
            // at the end).  The largest row sum seen is kept instead (one instruction); if it shows,
            // when the item's steps are done, that some scores outgrew the reference by 2^64 or
            // overflowed, the wavefront recomputes its rows the careful way (see below).  The maximum,
            // its exchange between the half-waves and the comparison were a sixth of this loop's
            // vector instructions, and those are what bounds it.
            float psum = 0.f, pprev = 0.f;
            const float moff = m_run * a.scale_l2;
#pragma unroll
            for (int j = 0; j < NSLOT; j++) {
                if (j + AH < NSLOT) fr[j + AH] = rd(j + AH);
                if (j < KS) {
                    sn = mfma32(fr[j], qf[j < KS ? j : 0], sn);
                } else {
                    const int st = (j - KS) / DB;
                    Frag8 pf;
                    pf.u = u32x4{pp[4 * st], pp[4 * st + 1], pp[4 * st + 2], pp[4 * st + 3]};
                    oacc[(j - KS) % DB] = mfma32(fr[j], pf.v, oacc[(j - KS) % DB]);
                }
                if (PF && (HALVES == 2 || (j & 1))) {
                    const int n = HALVES == 2 ? j : j >> 1;
                    if (n < NCP / 2)
                        copy_one(mine + (KB ^ 1) * TILE, kbase + (int64_t)(t + 2) * kFwdBk * a.k_st, a.k_st, goffk, n);
                    else
                        copy_one(mine + (BUFS + (VB ^ 1)) * TILE, vbase + (int64_t)(t + 1) * kFwdBk * a.v_st, a.v_st, goffv, n - NCP / 2);
                }
                {
                    constexpr int NE = NSLOT;  // every slot carries its share of the 16 exponentials
#pragma unroll
                    for (int e = (j * 16) / NE; e < ((j + 1) * 16) / NE; e++) {
                        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e], a.scale_l2, -moff));
                        psum += p;
                        if (e & 1) {
                            pk[CP][e >> 1] = pack_bf16x2(pprev, p);
                            // keeps the arithmetic of this pair here: the optimiser would otherwise sink
                            // it to the pair's first use, below the matrix instructions it is to overlap
                            asm volatile("" : "+v"(pk[CP][e >> 1]));
                        } else {
                            pprev = p;
                        }
                    }
                }
            }
            asm volatile("" : "+v"(psum));  // the row-sum additions stay above, among the matrix instructions
            l_run += psum;
            psum_max = fmaxf(psum_max, psum);
        };

        // ---------------- pipeline fill: K tile 0 -> S(0), then iteration 0 --------------------
        // (the Q rows pass through this wavefront's quarter of the V buffers, which are idle until the
        // barrier: V tile 0 is requested after it)
        qrows.fragments(smem + BUFS * TILE + wave * (32 * L::ROWB), half * (REGION / L::ROWB), lo, qf, lane);
        wait_vmem();
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the fragments are in registers
        __syncthreads();
        // (short items draw their ticket here, long ones near their end: see window())
        const int draw_t = ntiles >= kLateTicketSteps ? ntiles - 2 : -1;
        if (draw_t < 0) deal.prefetch();
        if constexpr (BUFS == 2) {
            if (ntiles > 1) prefetch_k(1, 1);
            if (HALVES == 1 || ntiles > 0) prefetch_v(0, 0);
        }
        if (cmax >= 0) scores(sacc[0], smem);
        iter_slow(ic<0>{}, 0, smem + 32 * L::ROWB, smem);

        // ---------------- window t: iterations 2t+1 and 2t+2 ------------------------------------
        // (BUFS = 1: the tiles of window t, asked for when everybody is done with those before)
        auto fetch_now = [&](int t) {
            __syncthreads();
            if (t + 1 < ntiles) prefetch_k(t + 1, 0);
            prefetch_v(t, 0);
        };
        // Steady state: both iterations pipelined, and the copies of K tile t+2 and V tile t+1 (both
        // wholly inside the sequence) ride along with iteration 2t+1.  No branch but the rare rescale.
        auto window_steady = [&](auto vbc, int t) {
            constexpr int VB = decltype(vbc)::value, KB = BUFS == 2 ? VB ^ 1 : 0;  // V tile t in VB, K tile t+1 in KB
            lo.pin();
            if constexpr (BUFS == 1) fetch_now(t);
            wait_vmem();      // this wavefront's share of K tile t+1 and V tile t has landed
            __syncthreads();  // everybody's has, and everybody is done with K tile t and V tile t-1
            iter_fast(ic<1>{}, ic<KB>{}, ic<VB>{}, ic<BUFS == 2>{}, t);
            iter_fast(ic<0>{}, ic<KB>{}, ic<VB>{}, ic<0>{}, t);
        };
        // General form (pipeline fill and drain, masked block, ragged last tile): the copies go out in
        // one go after the barrier and the stages of an iteration run one after the other.  One copy
        // of the code for both buffer parities: the tile addresses are run-time values here.
        auto window = [&](int t) {
            const int vb = BUFS == 2 ? t & 1 : 0, kb = BUFS == 2 ? vb ^ 1 : 0;  // V tile t in vb, K tile t+1 in kb
            lo.pin();
            if constexpr (BUFS == 1) fetch_now(t);
            wait_vmem();      // this wavefront's share of K tile t+1 and V tile t has landed
            __syncthreads();  // everybody's has, and everybody is done with K tile t and V tile t-1
            if constexpr (BUFS == 2) {
                if (t + 2 < ntiles) prefetch_k(t + 2, kb ^ 1);
                if (t + 1 < ntiles) prefetch_v(t + 1, vb ^ 1);
            }
            // The ticket of the item after a LONG one is drawn in the item's last window but one: late enough
            // that the workgroup commits itself to another item only a few microseconds before it is
            // free for it (a ticket drawn when the item starts reserves the then-largest item for the
            // whole length of this one, and at the end of a pass every workgroup still owes an item
            // while others idle), early enough that the counter's round trip is over when the epilogue
            // is.  An item of a few steps gains nothing from that and pays the wait for the answer at its
            // end, so it draws right after its first barrier (behind its first loads, not in front of
            // them: answers come back in request order).
            if (t == draw_t) deal.prefetch();
            const char *sK = smem + kb * TILE, *sV = smem + (BUFS + vb) * TILE;
            iter_slow(ic<1>{}, 2 * t + 1, sK, sV);
            iter_slow(ic<0>{}, 2 * t + 2, sK + 32 * L::ROWB, sV + 32 * L::ROWB);
        };
        // windows [0, tsteady) are steady ones: t + 3 <= ntiles, (t + 3) * kFwdBk <= s, 2t + 3 <= cmax
        // (SHARD: and the blocks of a steady window lie before the first masked one)
        const int tsteady = max(0, min(min(ntiles, sk / kFwdBk) - 2, ((SHARD ? min(cmax, cmask) : cmax) - 1) >> 1));
        int t = 0;
        for (; t + 1 < tsteady; t += 2) {
            window_steady(ic<0>{}, t);
            window_steady(ic<BUFS == 2>{}, t + 1);
        }
        for (; t < ntiles; t++) window(t);

        // ---------------- (rare) the careful way, per wavefront ----------------------------------
        // Some row sum of a fast iteration was 2^64 or more, infinite or not a number: scores that
        // outgrew the reference such an iteration does not update.  The wavefront then computes its
        // 32 rows again, every block against its own maximum, on its own: K and V blocks of 32 keys
        // come straight from global memory through this wavefront's quarter of the K buffers (no
        // wavefront reads a K tile after the last window's barrier, and this one is past it).
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(psum_max < 0x1p64f)) != 0, 0)) {
            char *block = smem + wave * (32 * L::ROWB);
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
                for (int i = 0; i < 16; i++) oacc[db][i] = 0.f;
            m_run = SHARD ? -1e30f : -INFINITY;
            l_run = 0.f;
            for (int c = 0; c <= cmax; c++) {
                RowBlock<D> blk;
                blk.load(kbase, a.k_st, c * 32, sk - 1, lane);
                blk.stage(block, half * (REGION / L::ROWB), lane);
                f32x16 &sa = sacc[0];
                scores(sa, block);
                if (SHARD ? c >= cmask : c == cmask) {
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        const int kv = c * 32 + 8 * (i >> 2) + 4 * hl + (i & 3);
                        if (kv > lim) sa[i] = -INFINITY;
                    }
                }
                const float m_new = reference(block_max(sa));
                const float mo = m_new * a.scale_l2;
                float ps = 0.f;
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sa[i], a.scale_l2, -mo));
                    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sa[i + 1], a.scale_l2, -mo));
                    ps += p0 + p1;
                    pk[0][i >> 1] = pack_bf16x2(p0, p1);
                }
                blk.load(vbase, a.v_st, c * 32, sk - 1, lane);
                blk.stage(block, half * (REGION / L::ROWB), lane);  // (after the reads of the K block: one wavefront's LDS instructions execute in order)
                finish_block(m_new, ps);   // O and the row sum move to the block's reference first
                pv(pk[0], block);
            }
        }

        // ---- epilogue: normalise, write O (bf16) and LSE (natural log)
        KernArgs &e = fresh(args);
        float l_tot = halves_sum(l_run);
        if constexpr (HALVES == 2) {
            for (int t = ntiles * (3 - BUFS); t < windows * (3 - BUFS); t++) __syncthreads();  // (BUFS = 1: two a window)
            // the second half's O (not normalised), row maximum and row sum, through its own tiles' LDS
            __syncthreads();  // (everybody is done with them)
            f32x4 *const box = (f32x4 *)(smem + REGION) + wave * (DB * 4 * 64) + lane;
            float *const st = stats + 2 * (wave * 64 + lane);
            if (half) {
#pragma unroll
                for (int db = 0; db < DB; db++)
#pragma unroll
                    for (int i4 = 0; i4 < 4; i4++)
                        box[(db * 4 + i4) * 64] = f32x4{oacc[db][4 * i4], oacc[db][4 * i4 + 1], oacc[db][4 * i4 + 2], oacc[db][4 * i4 + 3]};
                st[0] = m_run;
                st[1] = l_tot;
            }
            __syncthreads();
            if (half) continue;
            const float m1 = st[0], M = fmaxf(m_run, m1);
            const float w0 = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run - M) * e.scale_l2);
            const float w1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m1 - M) * e.scale_l2);
            l_tot = w0 * l_tot + w1 * st[1];
            m_run = M;
            f32x4 o1[DB * 4];
#pragma unroll
            for (int i = 0; i < DB * 4; i++) o1[i] = box[i * 64];
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
                for (int i = 0; i < 16; i++) oacc[db][i] = w0 * oacc[db][i] + w1 * o1[db * 4 + i / 4][i % 4];
        }
        if constexpr (HALVES == 1) {  // (no list of halves has cut tiles, and here half of the wavefronts have left)
            if (nparts > 1) {
                // hand over (O unnormalised, row maximum, row sum); the part that arrives last merges
                // all parts in part order: O = sum_p 2^((m_p - M) scale_l2) O_p, likewise the row sums
                const int tid_ = wave * 64 + lane;  // (recomputed: keeping threadIdx alive through the tile loop costs a register)
                char *rec = e.pq.split_scratch + (int64_t)(slot + part) * kPartialBytes;
                split_store<DB>(rec, oacc, tid_);
                split_put((float *)(rec + 64 * kThreads * 4) + 2 * tid_, m_run);
                split_put((float *)(rec + 64 * kThreads * 4) + 2 * tid_ + 1, l_tot);
                if (!split_arrive(e.pq.split_flags + slot, nparts, &split_word, tid_)) continue;
                // all parts' row statistics first (one trip to memory for the lot), then the records in turn
                float mp[kMaxParts], lp[kMaxParts];
#pragma unroll
                for (int p = 0; p < kMaxParts; p++) {
                    const float *st = (const float *)(e.pq.split_scratch + (int64_t)(slot + min(p, nparts - 1)) * kPartialBytes +
                                                      64 * kThreads * 4) + 2 * tid_;
                    mp[p] = split_get(st);
                    lp[p] = split_get(st + 1);
                }
                float M = -INFINITY;
#pragma unroll
                for (int p = 0; p < kMaxParts; p++) M = p < nparts ? fmaxf(M, mp[p]) : M;
#pragma unroll
                for (int db = 0; db < DB; db++)
#pragma unroll
                    for (int i = 0; i < 16; i++) oacc[db][i] = 0.f;
                l_tot = 0.f;
#pragma unroll
                for (int p = 0; p < kMaxParts; p++) {
                    if (p < nparts) {
                        const float w = mp[p] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mp[p] - M) * e.scale_l2);
                        split_sum<DB>(e.pq.split_scratch + (int64_t)(slot + p) * kPartialBytes, oacc, w, tid_);
                        l_tot += w * lp[p];
                    }
                }
                m_run = M;
            }
        }
        if constexpr (SHARD) {
            if (e.dq) {
                // Fold into the fp32 running result of a ring instead of writing this shard's own O and LSE:
                // (o_acc, lse_acc) <- merge((o_acc, lse_acc), (O, LSE)), the row's two half-wave lanes each
                // taking their head-dim elements of the row; a part that counts nothing is silenced even
                // if it holds rubbish (a running result is started with lse_acc = -inf over anything).
                if (wq_lo < s) {
                    const int nrows = min(32, s - wq_lo);
                    float *const rows = (float *)e.dq + (tok0 + wq_lo) * e.dq_st + (int64_t)h * e.dq_sh;
                    RowsF32<DB> acc32;
                    int lane_ = lane;
                    asm volatile("" : "+v"(lane_));  // (address arithmetic stays in the epilogue)
                    lane_ &= 63;
                    acc32.load(rows, e.dq_st, nrows, lane_);
                    const int64_t li = (int64_t)h * e.T + tok0 + min(qrow, s - 1);
                    const float la = e.delta_out[li];
                    const float lb = l_tot > 0.f ? m_run * e.scale + __logf(l_tot) : -INFINITY;
                    const float m = fmaxf(la, lb);
                    float wa = 0.f, wb = 0.f, lse = -INFINITY;
                    if (m > -INFINITY) {
                        const float ea = __expf(la - m), eb = __expf(lb - m);
                        const float inv = 1.0f / (ea + eb);
                        wa = ea * inv;
                        wb = l_tot > 0.f ? eb * inv / l_tot : 0.f;  // (with the row's normalisation)
                        lse = m + __logf(ea + eb);
                    }
                    uint16_t *const o16 = e.out_o ? e.out_o + (tok0 + wq_lo) * e.o_st + (int64_t)h * e.o_sh : nullptr;  // the merged rows rounded to bf16, if asked for
                    acc32.each(smem + wave * (32 * L::ROWB), 32, oacc, wb, lane_, [&](int half, int n, int row, int col, f32x4 w) {
                        const float wr = __shfl(wa, row);  // the weight of the piece's row
                        const f32x4 o = acc32.old[half][n];
#pragma unroll
                        for (int i = 0; i < 4; i++) w[i] += wr > 0.f ? wr * o[i] : 0.f;
                        if (row < nrows) {
                            *(f32x4 *)(rows + (int64_t)row * e.dq_st + col) = w;
                            if (o16) *(u32x2 *)(o16 + (int64_t)row * e.o_st + col) = u32x2{pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3])};
                        }
                    });
                    if (qrow < s && hl == 0) e.delta_out[li] = lse;  // (after both lanes of the row have read it: one wavefront)
                }
                continue;
            }
        }
        if (qrow < s && hl == 0) e.lse_out[(int64_t)h * e.T + tok0 + qrow] = m_run * e.scale + __logf(l_tot);
        // O is staged through the K buffers without a barrier: no wavefront reads a K tile after the
        // barrier of the last window (the scores of the last blocks were issued in the window before),
        // and this wavefront is past that barrier, so every wavefront has reached it
        if (wq_lo < s)
            store_rowT_bf16_lds<DB>(smem + wave * (32 * L::ROWB), e.out_o + (tok0 + wq_lo) * e.o_st + (int64_t)h * e.o_sh,
                                    e.o_st, min(32, s - wq_lo), oacc,
                                    (SHARD && !(l_tot > 0.f)) ? 0.f : 1.0f / l_tot, lane);
        // deal.advance() holds the barrier after which the LDS buffers are reused by the next item
    }
    if constexpr (SEARCH) deal.finish_shared(); else deal.finish();
}

}  // namespace
}  // namespace flexsp
