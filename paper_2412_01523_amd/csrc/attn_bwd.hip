// Backward of packed causal attention (gradient of paper Sec. 2.1.2, Eq. 3, per sequence
// of the packed stream) for gfx950.  With P = softmax(scale Q K^T) recomputed from the saved
// log-sum-exp, and delta_i = dO_i . O_i:
//     dV = P^T dO,   dP = dO V^T,   dS = P o (dP - delta),
//     dQ = scale dS K,   dK = scale dS^T Q.
// Two kernels, no floating-point atomics (results are deterministic):
//   dQ      runs first; one work item = 128 query rows of one (sequence, head); loops over key
//           tiles; its prologue also computes delta and the base-2 log-sum-exp of its rows and
//           leaves them in the plan's scratch for the second kernel;
//   dK/dV   one work item = 64 keys of one (sequence, kv head); loops over the query heads of
//           the group and over the query rows that see those keys; dK^T, dV^T stay in
//           registers, so grouped-query heads are summed without a reduction pass.
// With D = 64 and long enough walks a dK/dV item is 128 keys (attn_bwd_dkv_wide_kernel).
// Small backwards run both as one launch (attn_bwd_both_kernel); the dK/dV pass then forms delta itself.  Large ones with D = 128 do not come
// here (attn_bwd_chain.hip).
// The 32x32 accumulator keeps one COLUMN per lane, and only its ROW index can be contracted
// in a following MFMA.  Hence dK/dV computes S = Q K^T (rows = queries) and dQ computes
// S^T = K Q^T (rows = keys).  Operands whose contraction index runs along the rows of a
// row-major LDS tile are fetched with the LDS transpose read.
#include <type_traits>

#include "attn_common.h"

namespace flexsp {
namespace {

// LDS fragments are read this many matrix instructions ahead of the one that uses them (the file is
// compiled in source order, like the forward kernel: the schedulers would sink the reads back)
constexpr int kReadAhead = 4;


template <int D>
constexpr int dkv_lds()  // bytes of LDS of the dK/dV pass: two steps (Q | dO | 64 log-sum-exp, 64 delta), four exchange slots
{
    return 2 * (2 * kDkvBq * LdsTile<D>::ROWB + 512) + 4 * 2048;
}
template <int D>
constexpr int dq_lds()  // ... of the dQ pass: two steps (K | V)
{
    return 4 * kDqBk * LdsTile<D>::ROWB;
}

// ------------------------------------------------------------------------------ dK / dV
// One work item = 64 keys of one (sequence, kv head).  The accumulators of 32 keys x D for both
// dK and dV, next to the K and V fragments, would take more than half of the register file and
// leave one wavefront per SIMD with nothing to hide its LDS latencies behind.  So TWO wavefronts
// share each block of 32 keys: per step of 64 query rows, wavefront j of the pair computes
// S = Q K^T, dP = dO V^T, P and dS for query block j only; then wavefront 0 accumulates
// dV^T += dO^T P and wavefront 1 accumulates dK^T += Q^T dS, each over BOTH query blocks.  For
// the other block each needs one bf16 fragment set from its partner (P one way, dS the other),
// swapped through LDS: a fragment is written and read back by the same lane numbers, so the swap
// is a plain linear copy.  No matrix work is duplicated, every wavefront fits in 256 registers,
// and two workgroups share a CU.
//
// SHARD = true is the variant for one shard of the keys (context parallelism; see the forward kernel):
// an item names 64 keys of the shard and the query rows of its sequence on this device, key j is
// visible to query row i iff j <= i + shift, the rows' log-sum-exp and delta are those of the COMPLETE
// attention, and the gradients may be added to what dK / dV hold.  Part p of a tile cut into k parts walks the p-th k-th of its steps.
//
// SELF = true: the log-sum-exp read is the forward's own and the workgroup forms delta = dO . O of a step's rows itself,
// from pieces of O requested with the step's tiles and the tile's own dO, so that the pass does not have to come after the dQ pass.
template <int D, bool SHARD, bool SELF>
__device__ __forceinline__ void dkv_pass(KernArgs &args, KernQueues &queues, const int first_wg, char *const smem, int &deal_word, int &split_word)
{
    typedef LdsTile<D> L;
    constexpr int KS = D / 16;
    constexpr int DB = D / 32;
    constexpr int BQ = kDkvBq;                  // query rows per step: two 32-row blocks
    constexpr int QTILE = BQ * L::ROWB;
    constexpr int STEP = 2 * QTILE + 512;       // Q | dO | lse2[64] delta[64]
    constexpr int XSLOT = 2048;                 // one 32 x 32 bf16 block (P or dS)
    static_assert(dkv_lds<D>() == 2 * STEP + 4 * XSLOT, "LDS of the pass");
    char *const exch = smem + 2 * STEP;

    const int tid = thread_id();
    const int lane0 = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = wave >> 1, j = wave & 1;     // key block; role: 0 accumulates dV, 1 accumulates dK
    LaneOffsets<D> lo;
    lo.init(lane0);
    // What depends on the wavefront's role is folded into the per-lane offsets once: phase 1 reads the
    // rows of query block j, phase 2 reads the dO tile (role 0) or the Q tile (role 1).  Every LDS
    // read of a step is then "offset register + compile-time constant", with no address arithmetic.
#pragma unroll
    for (int ks = 0; ks < KS; ks++) lo.nat[ks] += j * 32 * L::ROWB;
#pragma unroll
    for (int db = 0; db < DB; db++) {
        lo.tr[db][0] += j ? 0 : QTILE;
        lo.tr[db][1] += j ? 0 : QTILE;
    }
    ItemDealer deal;

    for (int item = deal.first(queues, args.grid, first_wg, &deal_word, wave, lane0); item >= 0; item = deal.advance()) {
        KernArgs &a = fresh(args);
        KernQueues &pq = fresh(queues);
        // s: query rows of the sequence; sk: its keys; sh: position of the first query minus position of
        // the first key (0 unless SHARD); tok0 / ktok0: their first rows in q, dO / k, v
        int s, sk, sh, g, kv0, first, total, nparts, part, slot, qfirst, nsteps;
        int64_t tok0, ktok0;
        if constexpr (SHARD) {
            const flexsp_shard_item it = load_shard_item((const flexsp_shard_item *)pq.items, item);
            s = it.q_len; sk = it.k_len; sh = it.shift; g = it.head_parts & 0xffff; kv0 = it.tile * kDkvBk;
            tok0 = it.q_start; ktok0 = it.k_start;
            // the first query row that sees the tile's first key, rounded down to a step boundary; no
            // steps at all when no row of the device sees these keys
            qfirst = a.causal ? (max(0, kv0 - sh) & ~(BQ - 1)) : 0;
            nsteps = max(0, (s - qfirst + BQ - 1) / BQ);
            first = 0; total = nsteps * a.G;
            part = (it.head_parts >> 16) & 0xff; nparts = it.head_parts >> 24; slot = it.slot;
            if (nparts > 1) {
                const int all = total;
                first = part * all / nparts;
                total = (part + 1) * all / nparts;
            }
        } else {
            const flexsp_item it = load_item(pq.items, item);
            s = it.seq_len; sk = s; sh = 0; g = it.head; kv0 = it.tile * kDkvBk;
            tok0 = it.seq_start; ktok0 = tok0;
            qfirst = a.causal ? kv0 : 0;  // kv0 is a multiple of BQ
            nsteps = (s - qfirst + BQ - 1) / BQ;
            // the item walks steps `first` .. `total`-1 of the tile's nsteps * G (all of them unless the tile was cut)
            first = it.step_begin; total = it.step_end;
            nparts = it.parts & 0xffff; part = it.parts >> 16; slot = it.slot;
        }
        // opaque per-item copy of the lane id: per-lane address arithmetic of an item stays inside
        // the item instead of being hoisted out of this loop into long-lived registers
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        lane &= 63;  // (its range is known again: divisions by the pieces of a row are shifts)
        const int r = lane & 31, hl = lane >> 5;
        const int wk_lo = kv0 + kb * 32;
        const int kvrow = wk_lo + r;  // this lane's key (column of S)

        const uint32_t goffq = tile_goff<D>(a.q_st, wave, lane), goffg = tile_goff<D>(a.do_st, wave, lane);
        // Steps are counted from the item's first one (n of them); which head and which query rows a step
        // covers is carried along instead of being divided out of a step number: (h_cur, q_cur) for the
        // step being computed, (h_nxt, q_nxt) for the one whose tiles are fetched meanwhile.
        const int n = total - first;
        // The ticket of the item after this one: a short item draws it now, a long one when its steps are
        // done (see the forward kernel; here not inside the steps: any branch there costs this kernel
        // 1-2 %, and behind a long item the wait for the answer, what the epilogue does not cover of
        // it, does not show).
        if (n < kLateTicketSteps) deal.prefetch();
        const int q_end = qfirst + nsteps * BQ;
        int h_cur = g * a.G, q_cur = qfirst;
        if (!SHARD || first > 0) {  // (a shard's tile may have no steps)
            h_cur += first / nsteps;
            q_cur += first % nsteps * BQ;
        }
        int h_nxt = h_cur, q_nxt = q_cur;
        auto advance_nxt = [&]() {
            q_nxt += BQ;
            if (q_nxt >= q_end) {
                q_nxt = qfirst;
                h_nxt++;
            }
        };
        // SELF: the pieces of O that correspond to the pieces of dO this lane copies into the tile, and (wavefront 0) a row's log-sum-exp
        constexpr int NO = SELF ? BQ * L::CH / kThreads : 1;
        u32x4 o_raw[NO];
        float lse_raw = 0.f;
        const uint32_t goffo = SELF ? tile_goff<D>(a.o_st, wave, lane) : 0;
        auto prefetch = [&](int h, int qs, int buf) {
            char *base = smem + buf * STEP;
            const uint16_t *qb = a.q + tok0 * a.q_st + (int64_t)h * a.q_sh;
            const uint16_t *gb = a.dO + tok0 * a.do_st + (int64_t)h * a.do_sh;
            if (__builtin_expect(qs + BQ <= s, 1)) {  // whole tile inside the sequence
                load_tile_async_fast<D, BQ>(base, qb + (int64_t)qs * a.q_st, a.q_st, goffq, wave);
                load_tile_async_fast<D, BQ>(base + QTILE, gb + (int64_t)qs * a.do_st, a.do_st, goffg, wave);
            } else {
                load_tile_async<D, BQ>(base, qb, a.q_st, qs, s - 1, wave, lane);
                load_tile_async<D, BQ>(base + QTILE, gb, a.do_st, qs, s - 1, wave, lane);
            }
            const float *const lse = a.lse_in + (int64_t)h * a.T + tok0 + min(qs + lane, s - 1);
            if constexpr (SELF) {
                // (rows past the sequence read as zeros: nobody looks at their delta)
                const uint32_t rowb = (uint32_t)a.o_st * 2u;
                const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)(a.o + (tok0 + qs) * a.o_st + (int64_t)h * a.o_sh), 0, (int)(min(s - qs, BQ) * rowb), 0x00020000);
#pragma unroll
                for (int i = 0; i < NO; i++) o_raw[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, goffo, i * (kThreads / L::CH) * rowb, 0);
                if (wave == 0) lse_raw = *lse;
            } else if (wave < 2) {  // wavefront 0: lse2 of the 64 rows, wavefront 1: delta
                global_to_lds4(wave ? a.delta_in + (lse - a.lse_in) : lse, base + 2 * QTILE + wave * 256);
            }
        };
        // SELF: the log-sum-exp to base 2 and -delta of the step in buffer `buf`, left where the step reads them (after this wavefront's own
        // copies have landed: it reads its pieces of dO from the tile)
        auto put_delta = [&](int buf) {
            char *base = smem + buf * STEP;
            float *to = (float *)(base + 2 * QTILE);
            u32x4 g_raw[NO];
#pragma unroll
            for (int i = 0; i < NO; i++) g_raw[i] = *(const u32x4 *)(base + QTILE + (i * kThreads + wave * 64 + lane) * 16);
#pragma unroll
            for (int i = 0; i < NO; i++) {
                float d = 0.f;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t gw = g_raw[i][e], ow = o_raw[i][e];
                    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, gw), __builtin_bit_cast(bf16x2, ow), d, false);
                }
                d = group_sum<L::CH>(d);
                if (lane % L::CH == 0) to[64 + (i * kThreads + wave * 64 + lane) / L::CH] = -d;
            }
            // (SHARD: a row that saw no key anywhere has P = 0)
            if (wave == 0) to[lane] = SHARD && lse_raw == -INFINITY ? INFINITY : lse_raw * 1.4426950408889634f;
        };
        if (n > 0) prefetch(h_cur, q_cur, 0);
        advance_nxt();

        // K and V fragments of the pair's 32 keys (B operands: column = key, k = head dim), through
        // this wavefront's quarter of tile buffer 1, which is idle until step 0 requests step 1's tiles
        bf16x8 kf[KS], vf[KS];
        {
            RowBlock<D> krows, vrows;
            krows.load(a.k + ktok0 * a.k_st + (int64_t)g * a.k_sh, a.k_st, wk_lo, sk - 1, lane);
            vrows.load(a.v + ktok0 * a.v_st + (int64_t)g * a.v_sh, a.v_st, wk_lo, sk - 1, lane);
            // (this kernel's fragment offsets point at row block j of a tile: wavefronts 2kb and 2kb+1 use
            // the two halves of one 64-row stretch, so the stretch's address serves both)
            char *stretch = smem + STEP + kb * (64 * L::ROWB);
            krows.fragments(stretch, j * 32, lo, kf, lane);
            vrows.fragments(stretch, j * 32, lo, vf, lane);
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): in registers before step 0's barrier frees the buffer
        }
        f32x16 accT[DB];  // dV^T (role 0) or dK^T (role 1): rows = head dim, column = key
#pragma unroll
        for (int d = 0; d < DB; d++)
#pragma unroll
            for (int i = 0; i < 16; i++) accT[d][i] = 0.f;

        auto step_fn = [&](auto bufc, int step) {
            constexpr int BUF = decltype(bufc)::value;
            const char *sQ = smem + BUF * STEP;
            const char *sG = sQ + QTILE;
            const float *sL = (const float *)(sQ + 2 * QTILE);  // lse2[64], -delta[64]
            const int q_lo = q_cur;
            // a block (32 queries x the pair's 32 keys) is empty when it lies past the end of the
            // sequence or wholly above the diagonal; both wavefronts of a pair agree on that
            auto empty = [&](int qb) {
                const int lo_ = q_lo + qb * 32;
                return lo_ >= s || (a.causal && lo_ + 31 + sh < wk_lo);
            };
            lo.pin();
            wait_vmem();
            if constexpr (SELF) put_delta(BUF);
            __syncthreads();  // tile `step` is in LDS; the previous step's exchange slots are free
            // (the copies of the next tiles go out after phase 1's matrix instructions, not here: a
            // wavefront waits until its copy instructions are accepted, and behind the barrier that wait
            // would sit in front of matrix work that is ready to go; about 1 % on batches of short
            // sequences; the same move in the dQ kernel cost 2 %)

            // ---- phase 1: P and dS of query block j
            // (matrix phases run at raised wave priority, the arithmetic between them at the base one: when
            // both workgroups of a compute unit want the matrix pipe, the one already in a matrix phase
            // finishes it first instead of both crawling through it together; 2-3 % on this kernel)
            __builtin_amdgcn_s_setprio(2);
            uint32_t pp[8], dd[8];
            const int my_lo = q_lo + j * 32;
            if (!empty(j)) {
                // The dP accumulator starts at -delta of its rows (the scratch holds delta negated), so the
                // matrix instructions deliver dP - delta and the subtraction costs no vector instruction.
                f32x16 sacc, pacc;
#pragma unroll
                for (int i4 = 0; i4 < 4; i4++) {
                    const f32x4 d4 = *(const f32x4 *)(sL + 64 + j * 32 + 8 * i4 + 4 * hl);
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        sacc[4 * i4 + e] = 0.f;
                        pacc[4 * i4 + e] = d4[e];
                    }
                }
                {
                    // fragment n: k step n / 2 of the Q tile (n even) or the dO tile (n odd); read AH ahead
                    constexpr int AH = kReadAhead, N = 2 * KS;
                    bf16x8 fr[N];
                    auto rd = [&](int n) { return lds_nat((n & 1) ? sG : sQ, lo.nat[n >> 1]); };  // (rows of block j: see lo.nat above)
#pragma unroll
                    for (int n = 0; n < AH; n++) fr[n] = rd(n);
#pragma unroll
                    for (int n = 0; n < N; n++) {
                        if (n + AH < N) fr[n + AH] = rd(n + AH);
                        if (n & 1)
                            pacc = mfma32(fr[n], vf[n >> 1], pacc);
                        else
                            sacc = mfma32(fr[n], kf[n >> 1], sacc);
                    }
                }
                __builtin_amdgcn_s_setprio(0);
                if (__builtin_expect(step + 1 < n, 1)) prefetch(h_nxt, q_nxt, BUF ^ 1);
                // rows of the accumulator: query my_lo + 8*i4 + 4*hl + e
                const bool masked = (a.causal && my_lo + sh < wk_lo + 31) || (my_lo + 32 > s);
                auto probs = [&](auto maskc) {
                    constexpr bool MASK = decltype(maskc)::value;
#pragma unroll
                    for (int i4 = 0; i4 < 4; i4++) {
                        const f32x4 l4 = *(const f32x4 *)(sL + j * 32 + 8 * i4 + 4 * hl);
                        float p[4], ds[4];
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[4 * i4 + e], a.scale_l2, -l4[e]));
                            if (MASK) {
                                const int qr = my_lo + 8 * i4 + 4 * hl + e;
                                p[e] = ((a.causal && qr + sh < kvrow) || qr >= s) ? 0.f : p[e];
                            }
                            ds[e] = p[e] * pacc[4 * i4 + e];
                        }
                        pp[2 * i4] = pack_bf16x2(p[0], p[1]);
                        pp[2 * i4 + 1] = pack_bf16x2(p[2], p[3]);
                        dd[2 * i4] = pack_bf16x2(ds[0], ds[1]);
                        dd[2 * i4 + 1] = pack_bf16x2(ds[2], ds[3]);
                    }
                };
                if (masked)
                    probs(std::true_type{});
                else
                    probs(std::false_type{});
                // hand the partner what it accumulates: role 0 gives dS, role 1 gives P
                char *slot = exch + (kb * 2 + j) * XSLOT + lane * 16;
                *(u32x4 *)(slot) = j ? u32x4{pp[0], pp[1], pp[2], pp[3]} : u32x4{dd[0], dd[1], dd[2], dd[3]};
                *(u32x4 *)(slot + 1024) = j ? u32x4{pp[4], pp[5], pp[6], pp[7]} : u32x4{dd[4], dd[5], dd[6], dd[7]};
            }
            if (empty(j) && step + 1 < n) prefetch(h_nxt, q_nxt, BUF ^ 1);  // no phase 1: the copies go out here
            __syncthreads();  // the partner's fragments are visible
            __builtin_amdgcn_s_setprio(2);

            // ---- phase 2: role 0: dV^T += dO^T P, role 1: dK^T += Q^T dS, both query blocks
            const char *sX = sQ;  // (+ QTILE for role 0, inside lo.tr)
#pragma unroll
            for (int qb = 0; qb < 2; qb++) {
                if (empty(qb)) continue;
                Frag8 f[2];
                if (qb == j) {  // this wavefront's own block: from registers
                    f[0].u = j ? u32x4{dd[0], dd[1], dd[2], dd[3]} : u32x4{pp[0], pp[1], pp[2], pp[3]};
                    f[1].u = j ? u32x4{dd[4], dd[5], dd[6], dd[7]} : u32x4{pp[4], pp[5], pp[6], pp[7]};
                } else {        // the partner's block: from its slot
                    const char *slot = exch + (kb * 2 + qb) * XSLOT + lane * 16;
                    f[0].u = *(const u32x4 *)(slot);
                    f[1].u = *(const u32x4 *)(slot + 1024);
                }
                {
                    constexpr int AH = kReadAhead, N = 2 * DB;  // fragment n: query half n / DB, head-dim block n % DB
                    bf16x8 fr[N];
                    auto rd = [&](int n) {
                        const int rowoff = (qb * 32 + (n / DB) * 16) * L::ROWB;
                        return lds_tr(sX, rowoff + lo.tr[n % DB][0], rowoff + lo.tr[n % DB][1]);
                    };
#pragma unroll
                    for (int n = 0; n < AH; n++) fr[n] = rd(n);
#pragma unroll
                    for (int n = 0; n < N; n++) {
                        if (n + AH < N) fr[n + AH] = rd(n + AH);
                        accT[n % DB] = mfma32(fr[n], f[n / DB].v, accT[n % DB]);
                    }
                }
            }
            __builtin_amdgcn_s_setprio(0);
            h_cur = h_nxt;
            q_cur = q_nxt;
            advance_nxt();
        };
        for (int step = 0; step < n; step += 2) {
            step_fn(std::integral_constant<int, 0>{}, step);
            if (step + 1 < n) step_fn(std::integral_constant<int, 1>{}, step + 1);
        }
        KernArgs &e = fresh(args);
        KernQueues &eq = fresh(queues);
        if (n >= kLateTicketSteps) deal.prefetch();
        if (nparts > 1) {
            split_store<DB>(eq.split_scratch + (int64_t)(slot + part) * kPartialBytes, accT, tid);
            if (!split_arrive(eq.split_flags + slot, nparts, &split_word, tid)) continue;  // a later part finishes the tile
#pragma unroll
            for (int d = 0; d < DB; d++)
#pragma unroll
                for (int i = 0; i < 16; i++) accT[d][i] = 0.f;
            for (int p = 0; p < nparts; p++)
                split_sum<DB>(eq.split_scratch + (int64_t)(slot + p) * kPartialBytes, accT, 1.0f, tid);
        }

        // role 0 writes dV rows, role 1 writes dK rows (scaled)
        char *const out = (char *)(j ? e.dk : e.dv);
        const int64_t ost = j ? e.dk_st : e.dv_st, osh = j ? e.dk_sh : e.dv_sh;
        const float mul = j ? e.scale : 1.0f;
        if (wk_lo >= sk) continue;
        char *const stage = smem + (n & 1) * STEP + wave * (32 * L::ROWB);  // the Q/dO buffer the last step did not use (every wavefront is past its barriers)
        if (e.grad_f32) {
            float *const rows = (float *)out + (ktok0 + wk_lo) * ost + (int64_t)g * osh;
            RowsF32<DB> f;
            if (SHARD && (e.grad_f32 & 2))  // added to the partial sums the rows hold
                f.add(stage, rows, ost, min(32, sk - wk_lo), accT, mul, lane);
            else
                f.store(stage, rows, ost, min(32, sk - wk_lo), accT, mul, lane);
        } else {
            store_rowT_bf16_lds<DB>(stage,
                                    (uint16_t *)out + (ktok0 + wk_lo) * ost + (int64_t)g * osh, ost,
                                    min(32, sk - wk_lo), accT, mul, lane);
        }
        // deal.advance() holds the barrier after which the tiles and the exchange slots are reused
    }
    deal.finish();
}

template <int D, bool SHARD>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_bwd_dkv_kernel(const AttnArgs)
{
    KernArgs &a = kernel_args();
    __shared__ __attribute__((aligned(1024))) char smem[dkv_lds<D>()];
    __shared__ int deal_word, split_word;
    dkv_pass<D, SHARD, false>(a, a.pq, 0, smem, deal_word, split_word);
}

// ------------------------------------------------------------------------------ dK / dV, 128 keys
// The D = 64 kernel for all but short walks over the queries.  One work item = 128 keys of one (sequence, kv head).  With D = 64 the
// accumulators of 32 keys for both dK and dV, their K and V fragments and a block's S and dP fit 256 registers, so a wavefront
// does its 32 keys alone: nothing is swapped between wavefronts, a step has one barrier instead of two, each tile of Q and dO serves
// twice the keys, and with four step buffers a tile is asked for two steps before it is read.  A wavefront walks the query rows in
// blocks of 32 as the forward does: the matrix instructions of block c - 1's sums carry the arithmetic of block c between them, then
// come S and dP of block c + 1.
// The kernel of 64 keys spends its time waiting (no unit busy for more than 43 % of the cycles: its waves stand at the two
// barriers and for LDS).  Here the matrix unit is busy for 50 %, other waits fall from 27 to 21 % of the waves' time: 30 011 tokens, 12
// heads on 4, not causal 532 -> 465 us (counters on); forward and backward of 8 heads, 64 keys -> 128: 65 536 tokens
// causal in sequences of 16 384 4 710 -> 4 465 us, 4 096 1 324 -> 1 251, 1 024 451 -> 443, 512 299 -> 297, 256 241 -> 244; 32 768
// tokens not causal 4 096 1 228 -> 1 149, 1 024 351 -> 327, 256 144 -> 136.  Same bits where no tile is cut (parts begin elsewhere): the
// sums are formed in the same order.
// (D = 128 needs 390 registers, one wavefront per SIMD; two 64-key workgroups are as fast or faster.)
__global__ __launch_bounds__(kThreads, 2) void attn_bwd_dkv_wide_kernel(const AttnArgs)
{
    constexpr int D = 64;
    typedef LdsTile<D> L;
    constexpr int KS = D / 16, DB = D / 32, BQ = kDkvBq;
    constexpr int QTILE = BQ * L::ROWB;
    constexpr int STEP = 2 * QTILE + 512;  // Q | dO | lse2[64] delta[64]
    constexpr int NB = 4;                  // step buffers: two in use, two on their way
    constexpr int NCP = 2 * BQ * L::CH / kThreads;  // copy instructions of a wavefront per step, the row statistics apart
    static_assert(2 * DB * 16 * kThreads * 4 <= kPartialBytes, "a part's sums are one record");
    __shared__ __attribute__((aligned(1024))) char smem[NB * STEP];
    __shared__ int deal_word, split_word;
    KernArgs &args = kernel_args();
    KernQueues &queues = args.pq;

    const int tid = thread_id();
    const int lane0 = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    LaneOffsets<D> lo0;
    lo0.init(lane0);
    ItemDealer deal;

    for (int item = deal.first(queues, args.grid, 0, &deal_word, wave, lane0); item >= 0; item = deal.advance()) {
        KernArgs &a = fresh(args);
        const flexsp_item it = load_item(a.pq.items, item);
        const int s = it.seq_len, g = it.head, kv0 = it.tile * kDkvWideBk;
        const int64_t tok0 = it.seq_start;
        const int qfirst = a.causal ? kv0 : 0;
        const int nsteps = (s - qfirst + BQ - 1) / BQ;
        const int first = it.step_begin, n = it.step_end - first;
        const int nparts = it.parts & 0xffff, part = it.parts >> 16, slot = it.slot;
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        lane &= 63;
        const int r = lane & 31, hl = lane >> 5;
        const int wk_lo = kv0 + wave * 32;  // the wavefront's first key
        const int kvrow = wk_lo + r;        // this lane's key (column of S)
        const bool causal = a.causal != 0;
        const float scale_l2 = a.scale_l2;
        if (n < kLateTicketSteps) deal.prefetch();
        const int q_end = qfirst + nsteps * BQ;
        const uint32_t goffq = tile_goff<D>(a.q_st, wave, lane), goffg = tile_goff<D>(a.do_st, wave, lane);
        int h_f = g * a.G + first / nsteps, q_f = qfirst + (first % nsteps) * BQ;  // the step fetched next
        int buf_f = 0, left_f = n;
        int q_t = q_f;  // the step whose tile the window accumulates from
        auto next_q = [&](int q) { return q + BQ >= q_end ? qfirst : q + BQ; };
        auto fetch = [&]() {  // asks for the next step's tiles, if there is one
            if (left_f <= 0) return;
            char *base = smem + buf_f * STEP;
            const uint16_t *qb = a.q + tok0 * a.q_st + (int64_t)h_f * a.q_sh;
            const uint16_t *gb = a.dO + tok0 * a.do_st + (int64_t)h_f * a.do_sh;
            if (wave < 2) {  // wavefront 0: lse2 of the 64 rows, wavefront 1: delta
                const float *src = (wave ? a.delta_in : a.lse_in) + (int64_t)h_f * a.T + tok0 + min(q_f + lane, s - 1);
                global_to_lds4(src, base + 2 * QTILE + wave * 256);
            }
            if (__builtin_expect(q_f + BQ <= s, 1)) {
                load_tile_async_fast<D, BQ>(base, qb + (int64_t)q_f * a.q_st, a.q_st, goffq, wave);
                load_tile_async_fast<D, BQ>(base + QTILE, gb + (int64_t)q_f * a.do_st, a.do_st, goffg, wave);
            } else {
                load_tile_async<D, BQ>(base, qb, a.q_st, q_f, s - 1, wave, lane);
                load_tile_async<D, BQ>(base + QTILE, gb, a.do_st, q_f, s - 1, wave, lane);
            }
            left_f--;
            buf_f = buf_f + 1 == NB ? 0 : buf_f + 1;
            q_f += BQ;
            if (q_f >= q_end) {
                q_f = qfirst;
                h_f++;
            }
        };
        fetch();
        // K and V fragments of the wavefront's keys, through its quarter of the last buffer, which is idle until window 0
        bf16x8 kf[KS], vf[KS];
        {
            RowBlock<D> krows, vrows;
            krows.load(a.k + tok0 * a.k_st + (int64_t)g * a.k_sh, a.k_st, wk_lo, s - 1, lane);
            vrows.load(a.v + tok0 * a.v_st + (int64_t)g * a.v_sh, a.v_st, wk_lo, s - 1, lane);
            char *region = smem + (NB - 1) * STEP + wave * (32 * L::ROWB);
            krows.fragments(region, 0, lo0, kf, lane);
            vrows.fragments(region, 0, lo0, vf, lane);
            __builtin_amdgcn_s_waitcnt(0xC07F);
        }
        for (int i = 1; i < NB - 1; i++) fetch();
        f32x16 accV[DB], accK[DB];
#pragma unroll
        for (int d = 0; d < DB; d++) accV[d] = accK[d] = f32x16{};
        // block c = rows 32 * (c & 1) .. of step c / 2; S and dP - delta of the latest block in sa, pa, P and dS of block c in pp, dd[c & 1]
        f32x16 sa, pa;
        uint32_t pp[2][8], dd[2][8];
        asm volatile("" : "=v"(sa), "=v"(pa));
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int i = 0; i < 8; i++) asm volatile("" : "=v"(pp[j][i]), "=v"(dd[j][i]));
        // LDS addresses: in window t the scores read the tiles of step t + 1 (nat, st_n), the sums those of step t (tr, st_t)
        int nat[KS], tr[DB][2], st_n = hl * 16, st_t = hl * 16;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) nat[ks] = lo0.nat[ks];
#pragma unroll
        for (int db = 0; db < DB; db++) tr[db][0] = lo0.tr[db][0], tr[db][1] = lo0.tr[db][1];
        auto empty = [&](int q) { return wk_lo >= s || q >= s || (causal && q + 31 < wk_lo); };
        auto masked = [&](int q) { return (causal && q < wk_lo + 31) || q + 32 > s; };

        auto scores = [&](int half) {
#pragma unroll
            for (int i4 = 0; i4 < 4; i4++) {
                const f32x4 d4 = *(const f32x4 *)(smem + st_n + 2 * QTILE + 256 + half * 128 + 32 * i4);
#pragma unroll
                for (int e = 0; e < 4; e++) pa[4 * i4 + e] = d4[e];
            }
            constexpr int AH = kReadAhead, N = 2 * KS;
            bf16x8 fr[N];
            auto rd = [&](int i) { return lds_nat(smem, ((i & 1) ? QTILE : 0) + half * 32 * L::ROWB + nat[i >> 1]); };
#pragma unroll
            for (int i = 0; i < AH; i++) fr[i] = rd(i);
#pragma unroll
            for (int i = 0; i < N; i++) {
                if (i + AH < N) fr[i + AH] = rd(i + AH);
                if (i & 1)
                    pa = mfma32(fr[i], vf[i >> 1], pa);
                else
                    sa = mfma32(fr[i], kf[i >> 1], i ? sa : f32x16{});
            }
        };
        // q: the block's first row; stat: per-lane address of its step's row statistics
        auto probs = [&](uint32_t (&p8)[8], uint32_t (&d8)[8], int q, int stat, int half) {
            const bool mask = masked(q);
#pragma unroll
            for (int i4 = 0; i4 < 4; i4++) {
                const f32x4 l4 = *(const f32x4 *)(smem + stat + 2 * QTILE + half * 128 + 32 * i4);
                float p[4], ds[4];
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sa[4 * i4 + e], scale_l2, -l4[e]));
                    if (mask) {
                        const int qr = q + 8 * i4 + 4 * hl + e;
                        p[e] = ((causal && qr < kvrow) || qr >= s) ? 0.f : p[e];
                    }
                    ds[e] = p[e] * pa[4 * i4 + e];
                }
                p8[2 * i4] = pack_bf16x2(p[0], p[1]);
                p8[2 * i4 + 1] = pack_bf16x2(p[2], p[3]);
                d8[2 * i4] = pack_bf16x2(ds[0], ds[1]);
                d8[2 * i4 + 1] = pack_bf16x2(ds[2], ds[3]);
            }
        };
        auto sums = [&](const uint32_t (&p8)[8], const uint32_t (&d8)[8], int half) {
            constexpr int AH = kReadAhead, N = 4 * DB;
            bf16x8 fr[N];
            auto rd = [&](int i) {
                const int k = i >> 1, at = ((i & 1) ? 0 : QTILE) + (half * 32 + (k / DB) * 16) * L::ROWB;
                return lds_tr(smem, at + tr[k % DB][0], at + tr[k % DB][1]);
            };
#pragma unroll
            for (int i = 0; i < AH; i++) fr[i] = rd(i);
#pragma unroll
            for (int i = 0; i < N; i++) {
                if (i + AH < N) fr[i + AH] = rd(i + AH);
                const int k = i >> 1, o = 4 * (k / DB);
                Frag8 f;
                if (i & 1) {
                    f.u = u32x4{d8[o], d8[o + 1], d8[o + 2], d8[o + 3]};
                    accK[k % DB] = mfma32(fr[i], f.v, accK[k % DB]);
                } else {
                    f.u = u32x4{p8[o], p8[o + 1], p8[o + 2], p8[o + 3]};
                    accV[k % DB] = mfma32(fr[i], f.v, accV[k % DB]);
                }
            }
        };
        // sums of block c - 1 and, between their matrix instructions, the arithmetic of block c (its half CP of a tile; block c - 1 is the
        // other half)
        auto sums_probs = [&](auto cpc, int stat) {
            constexpr int CP = decltype(cpc)::value;
            constexpr int HALF = CP ? 0 : 1, AH = kReadAhead, N = 4 * DB;
            const uint32_t(&p8)[8] = pp[CP ^ 1], (&d8)[8] = dd[CP ^ 1];
            bf16x8 fr[N];
            f32x4 l4[4];
            auto rd = [&](int i) {
                const int k = i >> 1, at = ((i & 1) ? 0 : QTILE) + (HALF * 32 + (k / DB) * 16) * L::ROWB;
                return lds_tr(smem, at + tr[k % DB][0], at + tr[k % DB][1]);
            };
            l4[0] = *(const f32x4 *)(smem + stat + 2 * QTILE + CP * 128);
#pragma unroll
            for (int i = 0; i < AH; i++) fr[i] = rd(i);
            float p0 = 0.f, d0 = 0.f;
#pragma unroll
            for (int i = 0; i < N; i++) {
                if (i + AH < N) fr[i + AH] = rd(i + AH);
                if (i * 4 % N == 0 && i * 4 / N < 3) l4[i * 4 / N + 1] = *(const f32x4 *)(smem + stat + 2 * QTILE + CP * 128 + 32 * (i * 4 / N + 1));
                const int k = i >> 1, o = 4 * (k / DB);
                Frag8 f;
                if (i & 1) {
                    f.u = u32x4{d8[o], d8[o + 1], d8[o + 2], d8[o + 3]};
                    accK[k % DB] = mfma32(fr[i], f.v, accK[k % DB]);
                } else {
                    f.u = u32x4{p8[o], p8[o + 1], p8[o + 2], p8[o + 3]};
                    accV[k % DB] = mfma32(fr[i], f.v, accV[k % DB]);
                }
#pragma unroll
                for (int e = (i * 16) / N; e < ((i + 1) * 16) / N; e++) {
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sa[e], scale_l2, -l4[e >> 2][e & 3]));
                    const float ds = p * pa[e];
                    if (e & 1) {
                        pp[CP][e >> 1] = pack_bf16x2(p0, p);
                        dd[CP][e >> 1] = pack_bf16x2(d0, ds);
                        asm volatile("" : "+v"(pp[CP][e >> 1]), "+v"(dd[CP][e >> 1]));
                    } else {
                        p0 = p;
                        d0 = ds;
                    }
                }
            }
        };
        // Tile t + 1 has landed, everybody's share of it, and everybody is done with tile t - 1.  `later`: tile t + 2 is on its
        // way and may stay there: the NCP copies that were asked for last (behind its row statistics).
        static_assert(NCP == 4, "the wait below");
        auto settle = [&](bool later) {
            if (later)
                __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4)
            else
                wait_vmem();
            __syncthreads();
        };
        // fill: S, dP of blocks 0 and 1, P, dS of block 0
        settle(n > 2);  // (tile 0: tile 1 may be waited for as well)
        if (!empty(q_t)) {
            scores(0);
            probs(pp[0], dd[0], q_t, st_t, 0);
        }
        if (!empty(q_t + 32)) scores(1);
        int cur = 0;  // buffer of step t
        int t = 0, q_n = next_q(q_t), up;
        // Window t: P, dS of blocks 2 t + 1 and 2 t + 2, S, dP of blocks 2 t + 2 and 2 t + 3, the sums of blocks 2 t and 2 t + 1.
        auto enter = [&]() {
            up = cur + 1 == NB ? -(NB - 1) * STEP : STEP;  // from the buffer of step t to that of step t + 1
#pragma unroll
            for (int ks = 0; ks < KS; ks++) nat[ks] += up;
            st_n += up;
            settle(t + 2 < n);
            fetch();
        };
        auto leave = [&]() {
#pragma unroll
            for (int db = 0; db < DB; db++) tr[db][0] += up, tr[db][1] += up;
            st_t += up;
            cur = cur + 1 == NB ? 0 : cur + 1;
            q_t = q_n;
            q_n = next_q(q_n);
            t++;
        };
        while (t < n) {
            // windows from here on without an empty block and without a masked one among those whose arithmetic they do
            const int from = causal ? wk_lo + 31 : 0;  // first row from which a block is not masked
            int run = q_t + 32 < from || q_t + 64 > s || q_n < from || wk_lo >= s ? 0 : max(0, min(n - 1 - t, (s - q_n) / BQ));
            for (; run > 0; run--) {
                enter();
                sums_probs(std::integral_constant<int, 1>{}, st_t);
                scores(0);
                sums_probs(std::integral_constant<int, 0>{}, st_n);
                scores(1);
                leave();
            }
            if (t >= n) break;
            enter();
            const bool more = t + 1 < n;
            if (!empty(q_t)) sums(pp[0], dd[0], 0);
            if (!empty(q_t + 32)) {
                probs(pp[1], dd[1], q_t + 32, st_t, 1);
                sums(pp[1], dd[1], 1);
            }
            if (more && !empty(q_n)) {
                scores(0);
                probs(pp[0], dd[0], q_n, st_n, 0);
            }
            if (more && !empty(q_n + 32)) scores(1);
            leave();
        }
        KernArgs &e = fresh(args);
        if (n >= kLateTicketSteps) deal.prefetch();
        if (nparts > 1) {
            constexpr int HALF = DB * 16 * kThreads * 4;  // bytes of one of the two sums
            char *rec = e.pq.split_scratch + (int64_t)(slot + part) * kPartialBytes;
            split_store<DB>(rec, accV, tid);
            split_store<DB>(rec + HALF, accK, tid);
            if (!split_arrive(e.pq.split_flags + slot, nparts, &split_word, tid)) continue;  // a later part finishes the tile
#pragma unroll
            for (int d = 0; d < DB; d++) accV[d] = accK[d] = f32x16{};
            for (int p = 0; p < nparts; p++) {
                const char *from = e.pq.split_scratch + (int64_t)(slot + p) * kPartialBytes;
                split_sum<DB>(from, accV, 1.0f, tid);
                split_sum<DB>(from + HALF, accK, 1.0f, tid);
            }
        }
        if (wk_lo >= s) continue;
        char *const stage = smem + (n % NB) * STEP + wave * (32 * L::ROWB);  // (nobody reads this buffer after the last window's barrier)
        const int rows = min(32, s - wk_lo);
        auto put = [&](void *out, int32_t st, int32_t sh, const f32x16 (&acc)[DB], float mul) {
            if (e.grad_f32) {
                RowsF32<DB> f;
                f.store(stage, (float *)out + (tok0 + wk_lo) * st + (int64_t)g * sh, st, rows, acc, mul, lane);
            } else {
                store_rowT_bf16_lds<DB>(stage, (uint16_t *)out + (tok0 + wk_lo) * st + (int64_t)g * sh, st, rows, acc, mul, lane);
            }
        };
        put(e.dv, e.dv_st, e.dv_sh, accV, 1.0f);
        put(e.dk, e.dk_st, e.dk_sh, accK, e.scale);
    }
    deal.finish();
}

// ------------------------------------------------------------------------------ dQ
// SHARD = true: the rows' share of dQ that comes from one shard of the keys (see the dK/dV kernel): the
// log-sum-exp read here is that of the complete attention and `o` the complete output, so delta is the
// complete one; a part of a cut tile comes as an item of its own with its key range and shift.
template <int D, bool SHARD>
__device__ __forceinline__ void dq_pass(KernArgs &args, KernQueues &queues, const int first_wg, char *const smem, int &deal_word, int &split_word)
{
    typedef LdsTile<D> L;
    constexpr int KS = D / 16;
    constexpr int DB = D / 32;
    constexpr int TILE = kDqBk * L::ROWB;
    static_assert(dq_lds<D>() == 4 * TILE, "LDS of the pass");  // [buffer][K | V]

    const int tid = thread_id();
    const int lane0 = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    LaneOffsets<D> lo;
    lo.init(lane0);
    ItemDealer deal;

    for (int item = deal.first(queues, args.grid, first_wg, &deal_word, wave, lane0); item >= 0; item = deal.advance()) {
        KernArgs &a = fresh(args);
        KernQueues &pq = fresh(queues);
        // s: query rows of the sequence; sk: keys counted from the item's first one; rel: position of a
        // row among those keys minus its row index; tok0 / ktok0: first rows in q, o, dO / k, v
        int s, sk, rel, h, q0, ntiles, nparts, part, slot;
        int64_t tok0, ktok0;
        if constexpr (SHARD) {
            const flexsp_shard_item it = load_shard_item((const flexsp_shard_item *)pq.items, item);
            s = it.q_len; sk = it.k_len; rel = it.shift; h = it.head_parts & 0xffff; q0 = it.tile * kDqBq;
            tok0 = it.q_start; ktok0 = it.k_start;
            part = (it.head_parts >> 16) & 0xff; nparts = it.head_parts >> 24; slot = it.slot;
            const int kv_end = a.causal ? max(0, min(sk, q0 + kDqBq + rel)) : sk;  // keys some row of the tile sees
            ntiles = (kv_end + kDqBk - 1) / kDqBk;
        } else {
            const flexsp_item it = load_item(pq.items, item);
            s = it.seq_len; h = it.head; q0 = it.tile * kDqBq;
            tok0 = it.seq_start;
            // The item walks key tiles step_begin .. step_end-1 (all of them unless the tile was cut: then it
            // hands its partial dQ over).  From here on keys are counted from the item's first one: koff keys
            // are skipped, `sk` remain, and a row's own position among them is its row index minus koff.
            const int koff = it.step_begin * kDqBk;
            ntiles = it.step_end - it.step_begin; sk = s - koff; rel = -koff;
            ktok0 = tok0 + koff;
            nparts = it.parts & 0xffff; part = it.parts >> 16; slot = it.slot;
        }
        // opaque per-item copy of the lane id: per-lane address arithmetic of an item stays inside
        // the item instead of being hoisted out of this loop into long-lived registers
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        lane &= 63;  // (its range is known again: divisions by the pieces of a row are shifts)
        const int r = lane & 31, hl = lane >> 5;
        const int g = h / a.G;
        const uint16_t *kbase = a.k + ktok0 * a.k_st + (int64_t)g * a.k_sh;
        const uint16_t *vbase = a.v + ktok0 * a.v_st + (int64_t)g * a.v_sh;
        const uint32_t goffk = tile_goff<D>(a.k_st, wave, lane), goffv = tile_goff<D>(a.v_st, wave, lane);
        auto prefetch = [&](int t, int buf) {
            char *dk = smem + buf * 2 * TILE, *dv = dk + TILE;
            if (__builtin_expect((t + 1) * kDqBk <= sk, 1)) {  // whole tile inside the sequence
                load_tile_async_fast<D, kDqBk>(dk, kbase + (int64_t)t * kDqBk * a.k_st, a.k_st, goffk, wave);
                load_tile_async_fast<D, kDqBk>(dv, vbase + (int64_t)t * kDqBk * a.v_st, a.v_st, goffv, wave);
            } else {
                load_tile_async<D, kDqBk>(dk, kbase, a.k_st, t * kDqBk, sk - 1, wave, lane);
                load_tile_async<D, kDqBk>(dv, vbase, a.v_st, t * kDqBk, sk - 1, wave, lane);
            }
        };
        if (!SHARD || ntiles > 0) prefetch(0, 0);  // (a tile of a shard's queries may see none of its keys)

        const int qrow = q0 + wave * 32 + r;
        const int wq_lo = q0 + wave * 32;
        const int wq_rel = wq_lo + rel;  // the wavefront's first row, counted like the keys
        const bool qok = qrow < s;
        bf16x8 qf[KS], gf[KS];  // B operands: column = query row, k = head dim
        // delta = dO . O of the row (the backward's preprocessing step, done here because this kernel
        // has the row's dO in registers anyway): this lane's half of the row, then the other half-wave's
        float dpart = 0.f;
        {
            // the three row blocks are requested together and pass one after the other through this
            // wavefront's quarter of tile buffer 1, which is idle until step 0 requests tile 1
            RowBlock<D> qrows, grows, orows;
            qrows.load(a.q + tok0 * a.q_st + (int64_t)h * a.q_sh, a.q_st, wq_lo, s - 1, lane);
            grows.load(a.dO + tok0 * a.do_st + (int64_t)h * a.do_sh, a.do_st, wq_lo, s - 1, lane);
            orows.load(a.o + tok0 * a.o_st + (int64_t)h * a.o_sh, a.o_st, wq_lo, s - 1, lane);
            char *region = smem + 2 * TILE + wave * (32 * L::ROWB);
            bf16x8 of[KS];
            qrows.fragments(region, 0, lo, qf, lane);
            grows.fragments(region, 0, lo, gf, lane);
            orows.fragments(region, 0, lo, of, lane);
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): in registers before step 0's barrier frees the buffer
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
                Frag8 fg, fo;
                fg.v = gf[ks];
                fo.v = of[ks];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    // (scalars first: a bit cast applied to a vector element in place reads element 0)
                    const uint32_t gw = fg.u[i], ow = fo.u[i];
                    dpart = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, gw), __builtin_bit_cast(bf16x2, ow),
                                                            dpart, false);
                }
            }
        }
        const float delta = halves_sum(dpart);
        // The dP accumulator of every block starts at -delta of its column, so the matrix instructions deliver dP - delta: sixteen
        // registers of the same value, against a subtraction per score (67 -> 53 vector instructions for 24 matrix ones).  Forward and
        // backward, as a ratio to the same older build, without -> with: 30 011 tokens, 12 heads on 4, D = 64 1.052 -> 1.066; one sequence
        // of 131 072 tokens, 8 heads 1.000 -> 1.007; 49 152 tokens in short sequences 1.031 -> 1.037.  dQ's error against fp64 is the same
        // to five digits (1.69e-3 to 1.97e-3 over eight shapes).
        f32x16 minus_delta;
#pragma unroll
        for (int i = 0; i < 16; i++) minus_delta[i] = -delta;
        asm volatile("" : "+v"(minus_delta));  // (kept, not formed again in front of every block)
        // the log-sum-exp in base 2, so that the recomputation is one fma + exp2 per score; +inf makes
        // P = 0 for rows past the end of the sequence
        float lse2 = qok ? a.lse_in[(int64_t)h * a.T + tok0 + qrow] * 1.4426950408889634f : INFINITY;
        if constexpr (SHARD) lse2 = lse2 == -INFINITY ? INFINITY : lse2;  // a row that saw no key anywhere

        f32x16 dqT[DB];  // rows = head dim, column = query
#pragma unroll
        for (int db = 0; db < DB; db++)
#pragma unroll
            for (int i = 0; i < 16; i++) dqT[db][i] = 0.f;

        const int draw_t = ntiles >= kLateTicketSteps ? ntiles - 3 : 0;  // the step in which the next ticket is drawn
        auto step_fn = [&](auto bufc, int t) {
            constexpr int BUF = decltype(bufc)::value;
            const char *sK = smem + BUF * 2 * TILE;
            const char *sV = sK + TILE;
            const int kv0 = t * kDqBk;
            lo.pin();
            wait_vmem();
            __syncthreads();
            // the next item's ticket: three steps before a long item ends, in a short one's first step (see the forward kernel)
            if (t == draw_t) deal.prefetch();
            if (__builtin_expect(t + 1 < ntiles, 1)) prefetch(t + 1, BUF ^ 1);
            if (a.causal && kv0 > wq_rel + 31) return;

            const bool need_mask = SHARD ? ((a.causal && kv0 + kDqBk - 1 > wq_rel) || kv0 + kDqBk > sk)
                                         : (a.causal ? (kv0 + kDqBk - 1 > wq_rel) : (kv0 + kDqBk > sk));
            const int lim = SHARD ? (a.causal ? min(qrow + rel, sk - 1) : sk - 1) : (a.causal ? qrow + rel : sk - 1);
            // one 32-key block at a time (keeps the register count under half the file)
#pragma unroll
            for (int kb = 0; kb < 2; kb++) {
                if (a.causal && kv0 + kb * 32 > wq_rel + 31) continue;  // block wholly above the diagonal
                f32x16 sacc, pacc;
                {
                    constexpr int AH = kReadAhead, N = 2 * KS;  // fragment n: k step n / 2 of the K tile (n even) or the V tile (n odd)
                    bf16x8 fr[N];
                    auto rd = [&](int n) { return lds_nat((n & 1) ? sV : sK, kb * 32 * L::ROWB + lo.nat[n >> 1]); };
#pragma unroll
                    for (int n = 0; n < AH; n++) fr[n] = rd(n);
#pragma unroll
                    for (int n = 0; n < N; n++) {
                        if (n + AH < N) fr[n + AH] = rd(n + AH);
                        if (n & 1)
                            pacc = mfma32(fr[n], gf[n >> 1], n > 1 ? pacc : minus_delta);
                        else
                            sacc = mfma32(fr[n], qf[n >> 1], n ? sacc : f32x16{});
                    }
                }
                uint32_t dd[8];
                auto dsfn = [&](auto maskc) {
                    constexpr bool MASK = decltype(maskc)::value;
#pragma unroll
                    for (int i = 0; i < 16; i += 2) {
                        float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], a.scale_l2, -lse2));
                        float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i + 1], a.scale_l2, -lse2));
                        if (MASK) {
                            const int kv = kv0 + kb * 32 + 8 * (i >> 2) + 4 * hl + (i & 3);
                            p0 = kv > lim ? 0.f : p0;
                            p1 = kv + 1 > lim ? 0.f : p1;
                        }
                        dd[i >> 1] = pack_bf16x2(p0 * pacc[i], p1 * pacc[i + 1]);
                    }
                };
                if (need_mask)
                    dsfn(std::true_type{});
                else
                    dsfn(std::false_type{});
                // dQ^T += K^T dS^T
                {
                    constexpr int AH = kReadAhead, N = 2 * DB;  // fragment n: key half n / DB, head-dim block n % DB
                    bf16x8 fr[N];
                    auto rd = [&](int n) {
                        const int rowoff = (kb * 32 + (n / DB) * 16) * L::ROWB;
                        return lds_tr(sK, rowoff + lo.tr[n % DB][0], rowoff + lo.tr[n % DB][1]);
                    };
#pragma unroll
                    for (int n = 0; n < AH; n++) fr[n] = rd(n);
#pragma unroll
                    for (int n = 0; n < N; n++) {
                        if (n + AH < N) fr[n + AH] = rd(n + AH);
                        const int hf = n / DB;
                        Frag8 df;
                        df.u = u32x4{dd[4 * hf], dd[4 * hf + 1], dd[4 * hf + 2], dd[4 * hf + 3]};
                        dqT[n % DB] = mfma32(fr[n], df.v, dqT[n % DB]);
                    }
                }
            }
        };
        if (ntiles <= 0) deal.prefetch();
        for (int t = 0; t < ntiles; t += 2) {
            step_fn(std::integral_constant<int, 0>{}, t);
            if (t + 1 < ntiles) step_fn(std::integral_constant<int, 1>{}, t + 1);
        }

        KernArgs &e = fresh(args);
        KernQueues &eq = fresh(queues);
        // delta and the base-2 log-sum-exp are kept for the dK/dV kernel, which runs after this one (nowhere beside a
        // dK/dV pass in one launch: nobody would read them)
        // (stored here, not where they are computed: a store in flight there would be waited for by
        // the first tile's wait for its copy)
        if (e.delta_out && qok && hl == 0) {
            e.delta_out[(int64_t)h * e.T + tok0 + qrow] = -delta;  // negated: the dK/dV kernel starts its dP accumulator from it
            e.lse_out[(int64_t)h * e.T + tok0 + qrow] = lse2;
        }
        if (nparts > 1) {
            split_store<DB>(eq.split_scratch + (int64_t)(slot + part) * kPartialBytes, dqT, tid);
            if (!split_arrive(eq.split_flags + slot, nparts, &split_word, tid)) continue;  // a later part finishes the tile
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
                for (int i = 0; i < 16; i++) dqT[db][i] = 0.f;
            for (int p = 0; p < nparts; p++)
                split_sum<DB>(eq.split_scratch + (int64_t)(slot + p) * kPartialBytes, dqT, 1.0f, tid);
        }
        if (wq_lo >= s) continue;
        char *const stage = smem + (ntiles & 1) * 2 * TILE + wave * (32 * L::ROWB);  // the tile buffer the last step did not use (see the forward kernel)
        if (e.grad_f32) {
            float *const rows = (float *)e.dq + (tok0 + wq_lo) * e.dq_st + (int64_t)h * e.dq_sh;
            RowsF32<DB> f;
            if (SHARD && (e.grad_f32 & 2))  // added to the partial sum the rows hold
                f.add(stage, rows, e.dq_st, min(32, s - wq_lo), dqT, e.scale, lane);
            else
                f.store(stage, rows, e.dq_st, min(32, s - wq_lo), dqT, e.scale, lane);
        } else {
            store_rowT_bf16_lds<DB>(stage,
                                    (uint16_t *)e.dq + (tok0 + wq_lo) * e.dq_st + (int64_t)h * e.dq_sh, e.dq_st,
                                    min(32, s - wq_lo), dqT, e.scale, lane);
        }
        // deal.advance() holds the barrier after which the LDS buffers are reused by the next item
    }
    deal.finish();
}

template <int D, bool SHARD>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_bwd_dq_kernel(const AttnArgs)
{
    KernArgs &a = kernel_args();
    __shared__ __attribute__((aligned(1024))) char smem[dq_lds<D>()];
    __shared__ int deal_word, split_word;
    dq_pass<D, SHARD>(a, a.pq, 0, smem, deal_word, split_word);
}

// ------------------------------------------------------------------------------ both at once
// Small backwards, whose two passes have a workgroup per item each (see ItemDealer) and leave most of the chip idle:
// workgroups 0 .. dq_wg-1 run the dK/dV pass, the rest the dQ pass.  One launch less, and the passes' chains of
// memory trips and short steps run side by side instead of one after the other; the price is that the dK/dV pass reads
// O as well.  Forward and backward, two launches -> one: 635 tokens, 1 head 29.6 -> 22.2 us; 808 tokens, 4 heads 42.8 -> 31.7 us;
// 1 141 tokens, 16 heads on 2 94 -> 76 us; 5 630 tokens, 2 heads 45.0 -> 38.8 us.
// delta is formed from the piece of dO that the lane has just copied into the tile and the same piece of O, which waits for the step in
// a register: both rows in registers were 35 spilled ones with D = 128, and dO was fetched twice (1 201 tokens, 16 heads on 4 38.9 -> 37.8
// us; 5 630 tokens, 2 heads 51.0 -> 50.0).
// (A variant with the whole register file for launches of at most one workgroup per compute unit was worth 0.2 % over 156 drawn passes of up to
// 3e10 operations with D = 128, 1.6 % at the most, and nothing over 76 rings.)
template <int D, bool SHARD>
__global__ __launch_bounds__(kThreads, 2) void attn_bwd_both_kernel(const AttnArgs)
{
    KernArgs &a = kernel_args();
    constexpr int LDS = dkv_lds<D>() > dq_lds<D>() ? dkv_lds<D>() : dq_lds<D>();
    __shared__ __attribute__((aligned(1024))) char smem[LDS];
    __shared__ int deal_word, split_word;
    if (workgroup_id() >= a.dq_wg)
        dq_pass<D, SHARD>(a, a.dq_pq, a.dq_wg, smem, deal_word, split_word);
    else if (workgroup_id() < a.dkv_items)
        dkv_pass<D, SHARD, true>(a, a.pq, 0, smem, deal_word, split_word);
}

template <bool SHARD>
void start_both(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    launch(D == 64 ? attn_bwd_both_kernel<64, SHARD> : attn_bwd_both_kernel<128, SHARD>, a, grid, s);
}

}  // namespace

hipError_t launch_attn_bwd_dkv(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    if (a.chain) return launch_attn_bwd_chain(a, grid, s);
    if (a.wide)
        launch(attn_bwd_dkv_wide_kernel, a, grid, s);
    else if (a.dq_wg)
        start_both<false>(a, D, grid, s);
    else if (D == 128)
        launch(attn_bwd_dkv_kernel<128, false>, a, grid, s);
    else
        launch(attn_bwd_dkv_kernel<64, false>, a, grid, s);
    return hipGetLastError();
}

hipError_t launch_attn_bwd_dq(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    if (a.chain) return launch_attn_bwd_delta(a, s);
    if (D == 128)
        launch(attn_bwd_dq_kernel<128, false>, a, grid, s);
    else
        launch(attn_bwd_dq_kernel<64, false>, a, grid, s);
    return hipGetLastError();
}

hipError_t launch_attn_bwd_dkv_kvshard(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    if (a.dq_wg)
        start_both<true>(a, D, grid, s);
    else if (D == 128)
        launch(attn_bwd_dkv_kernel<128, true>, a, grid, s);
    else
        launch(attn_bwd_dkv_kernel<64, true>, a, grid, s);
    return hipGetLastError();
}

hipError_t launch_attn_bwd_dq_kvshard(const AttnArgs &a, int D, int grid, hipStream_t s)
{
    if (D == 128)
        launch(attn_bwd_dq_kernel<128, true>, a, grid, s);
    else
        launch(attn_bwd_dq_kernel<64, true>, a, grid, s);
    return hipGetLastError();
}

}  // namespace flexsp
