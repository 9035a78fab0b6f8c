// What the host decides about a launch and no entry point tells: csrc/flexsp_host.hip is part of this program, so its
// internals can be looked at.  Runs under AddressSanitizer and UndefinedBehaviorSanitizer with host-only contexts; the
// kernel launchers are stubs that fail.
#include <cstdio>
#include <cstdlib>

#include "flexsp_host.hip"

namespace flexsp {
hipError_t launch_pack(const void *, void *, int64_t, int, int, int, int, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_pack_many(int, const void *const *, void *const *, int64_t, const int32_t *, int, int, int, bool,
                            hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_fwd(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_fwd_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dkv(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dq(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dkv_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dq_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_lse_merge(const uint16_t *, const float *, const uint16_t *, const float *, uint16_t *, float *, int64_t,
                            int, int, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_lse_merge_acc(float *, float *, const uint16_t *, const float *, uint16_t *, int64_t, int, int, int32_t,
                                int32_t, int32_t, int32_t, int32_t, int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t static_scratch_init(int) { return hipErrorUnknown; }
}  // namespace flexsp

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAILED: %s (line %d)\n", #c, __LINE__); return 1; } } while (0)

// Tensors of a backward as consecutive dense blocks of one imagined address range (nothing is dereferenced).
struct Blocks {
    uintptr_t at = 1 << 20;
    uintptr_t take(int64_t bytes) { const uintptr_t p = at; at += (uintptr_t)bytes; return p; }
};

// One launch for both passes only where the outputs lie apart from the inputs.
static int check_overlap(flexsp_ctx *ctx)
{
    const int32_t cu[3] = {0, 300, 370}, cu_k[3] = {0, 200, 230}, shift[2] = {100, 40};
    const int Hq = 4, Hkv = 2, D = 64;
    for (int shard = 0; shard < 2; shard++)
        for (int f32 = 0; f32 < 2; f32++) {
            flexsp_plan *p = nullptr;
            if (shard)
                CHECK(flexsp_plan_create_kvshard(ctx, cu, cu_k, shift, 2, Hq, Hkv, D, 1, &p) == FLEXSP_OK);
            else
                CHECK(flexsp_plan_create(ctx, cu, 2, Hq, Hkv, D, 1, &p) == FLEXSP_OK);
            const int64_t T = cu[2], Tk = shard ? cu_k[2] : T, gb = f32 ? 4 : 2;
            AttnArgs a;
            std::memset(&a, 0, sizeof(a));
            a.grad_f32 = f32;
            Blocks m;
            const uintptr_t q = m.take(2 * T * Hq * D), o = m.take(2 * T * Hq * D), g = m.take(2 * T * Hq * D);
            const uintptr_t k = m.take(2 * Tk * Hkv * D), v = m.take(2 * Tk * Hkv * D), lse = m.take(4 * T * Hq);
            const uintptr_t dq = m.take(gb * T * Hq * D), dk = m.take(gb * Tk * Hkv * D), dv = m.take(gb * Tk * Hkv * D);
            a.q = (const uint16_t *)q; a.o = (const uint16_t *)o; a.dO = (const uint16_t *)g;
            a.k = (const uint16_t *)k; a.v = (const uint16_t *)v; a.lse_in = (const float *)lse;
            a.q_st = a.o_st = a.do_st = a.dq_st = Hq * D;
            a.k_st = a.v_st = a.dk_st = a.dv_st = Hkv * D;
            a.q_sh = a.o_sh = a.do_sh = a.dq_sh = a.k_sh = a.v_sh = a.dk_sh = a.dv_sh = D;
            auto apart = [&](uintptr_t dq_, uintptr_t dk_, uintptr_t dv_) {
                AttnArgs b = a;
                b.dq = (void *)dq_; b.dk = (void *)dk_; b.dv = (void *)dv_;
                return both_at_once(ctx, p, b) != 0;
            };
            CHECK(apart(dq, dk, dv));  // (and so the batch is one that the single launch takes)
            const int64_t rows = 2 * T * Hq * D, keys = 2 * Tk * Hkv * D;
            const uintptr_t inputs[] = {q, o, g, k, v, lse};
            const int64_t sizes[] = {rows, rows, rows, keys, keys, 4 * T * Hq};
            for (int i = 0; i < 6; i++) {
                const uintptr_t last = inputs[i] + sizes[i] - 16;  // an output that begins in the input's last 16 bytes ...
                CHECK(!apart(inputs[i], dk, dv) && !apart(dq, inputs[i], dv) && !apart(dq, dk, inputs[i]));
                CHECK(!apart(last, dk, dv) && !apart(dq, last, dv) && !apart(dq, dk, last));
                CHECK(!apart(inputs[i] - gb * T * Hq * D + 16, dk, dv));  // ... or ends in its first
            }
            CHECK(apart(dq, dk + 16, dv + 16));  // touching the range of no input
            flexsp_plan_destroy(p);
        }
    return 0;
}

// The list a pass of few items is launched with (one workgroup per item), which plan inspection does not show: every tile's
// steps exactly once, by one whole item or by parts with records of their own.
static int check_list(const flexsp_plan *p, int pass, const std::vector<std::vector<int64_t>> &tiles, int heads, int lowest)
{
    const HostPass &hp = p->pass[pass];
    size_t whole = 0;
    for (const auto &b : tiles) whole += b.size() * heads;
    if (hp.items.empty() || hp.items.size() > 512) {
        CHECK(hp.direct.empty());
        return 0;
    }
    const bool halves = pass == FLEXSP_PASS_FWD && p->halves;
    CHECK(halves ? hp.direct.size() == whole && whole <= (size_t)fwd_halves_room(p->D, 256) : hp.direct.size() >= whole && hp.direct.size() <= 512);
    std::vector<std::vector<std::vector<std::vector<flexsp_item>>>> of(tiles.size());
    for (size_t b = 0; b < tiles.size(); b++) of[b].assign(tiles[b].size(), std::vector<std::vector<flexsp_item>>(heads));
    for (const flexsp_item &it : hp.direct) {
        size_t b = 0;  // plans of shards name a sequence by its index, others by its first token
        if (p->kvshard)
            b = (size_t)it.seq_start;
        else
            while (b < tiles.size() && (p->cu[b] != it.seq_start || tiles[b].empty())) b++;
        CHECK(b < tiles.size() && it.tile >= 0 && (size_t)it.tile < tiles[b].size() && it.head >= 0 && it.head < heads);
        of[b][it.tile][it.head].push_back(it);
    }
    std::vector<char> taken((size_t)hp.records, 0);
    for (size_t b = 0; b < tiles.size(); b++)
        for (size_t t = 0; t < tiles[b].size(); t++)
            for (int h = 0; h < heads; h++) {
                std::vector<flexsp_item> &v = of[b][t][h];
                std::sort(v.begin(), v.end(), [](const flexsp_item &x, const flexsp_item &y) { return x.parts >> 16 < y.parts >> 16; });
                CHECK(!v.empty() && v[0].step_begin == 0 && v.back().step_end == tiles[b][t]);
                const int n = (int)v.size();
                CHECK(n <= kMaxParts);
                for (int i = 0; i < n; i++) {
                    CHECK(v[i].parts == ((i << 16) | n) && v[i].slot == v[0].slot);
                    CHECK(i == 0 || v[i].step_begin == v[i - 1].step_end);
                    CHECK(n == 1 || v[i].step_end - v[i].step_begin >= lowest);
                }
                CHECK((v[0].slot >= 0) == (n > 1));
                if (n > 1) {
                    CHECK(v[0].slot + n <= hp.records);
                    for (int i = 0; i < n; i++) CHECK(!taken[v[0].slot + i]++);
                }
            }
    return 0;
}

static int check_direct_lists(flexsp_ctx *ctx)
{
    unsigned seed = 4711;
    auto rnd = [&](int lo, int hi) { seed = seed * 1664525u + 1013904223u; return lo + (int)((seed >> 8) % (unsigned)(hi - lo + 1)); };
    int lists = 0, finer = 0, both = 0, halves = 0;
    for (int trial = 0; trial < 600; trial++) {
        const int Hkv = rnd(1, 4), G = rnd(0, 2) ? 1 : rnd(2, 8), Hq = Hkv * G, causal = rnd(0, 3) != 0;
        const int B = rnd(1, rnd(0, 1) ? 4 : 120), top = 1 << rnd(3, 12);
        std::vector<int32_t> cu(B + 1, 0), cu_k(B + 1, 0), shift(B, 0);
        for (int b = 0; b < B; b++) {
            cu[b + 1] = cu[b] + (rnd(0, 9) ? rnd(1, top) : 0);
            cu_k[b + 1] = cu_k[b] + (rnd(0, 9) ? rnd(1, 2 * top) : 0);
            shift[b] = rnd(-top, 2 * top);
        }
        for (int shard = 0; shard < 2; shard++) {
            flexsp_plan *p = nullptr;
            if (shard)
                CHECK(flexsp_plan_create_kvshard(ctx, cu.data(), cu_k.data(), shift.data(), B, Hq, Hkv, 128, causal, &p) == FLEXSP_OK);
            else
                CHECK(flexsp_plan_create(ctx, cu.data(), B, Hq, Hkv, 128, causal, &p) == FLEXSP_OK);
            std::vector<std::vector<int64_t>> rows(B), keys(B);  // steps of each sequence's query tiles and key tiles
            for (int b = 0; b < B; b++) {
                const int64_t sq = cu[b + 1] - cu[b], sk = shard ? cu_k[b + 1] - cu_k[b] : sq, sh = shard ? shift[b] : 0;
                for (int64_t t = 0; t * 128 < sq; t++) {
                    const int64_t seen = causal ? std::max<int64_t>(0, std::min(sk, (t + 1) * 128 + sh)) : sk;
                    rows[b].push_back((seen + 63) / 64 + shard);  // (a shard's tile without keys is still written)
                }
                for (int64_t t = 0; t * 64 < sk; t++) {
                    const int64_t first = causal ? std::max<int64_t>(0, t * 64 - sh) / 64 * 64 : 0;
                    keys[b].push_back(std::max<int64_t>(0, (sq - first + 63) / 64) * G + shard);
                }
            }
            for (int pass = 0; pass < 3; pass++) {
                const std::vector<std::vector<int64_t>> &steps = pass == FLEXSP_PASS_BWD_DKV ? keys : rows;
                const int heads = pass == FLEXSP_PASS_BWD_DKV ? Hkv : Hq;
                const HostPass &hp = p->pass[pass];
                if (pass == FLEXSP_PASS_FWD && p->halves) {  // (tiles of 64 rows)
                    CHECK(!shard && hp.records == 0);
                    std::vector<std::vector<int64_t>> rows64(B);
                    for (int b = 0; b < B; b++)
                        for (int64_t t = 0, sq = cu[b + 1] - cu[b]; t * 64 < sq; t++) rows64[b].push_back(((causal ? std::min(sq, (t + 1) * 64) : sq) + 63) / 64);
                    if (check_list(p, pass, rows64, heads, 0)) return 1;
                    halves++;
                } else if (check_list(p, pass, steps, heads, pass == FLEXSP_PASS_FWD ? kMinPartSteps : kShortPartSteps)) return 1;
                lists += !hp.direct.empty();
                finer += hp.direct.size() > hp.items.size();
            }
            AttnArgs a;
            std::memset(&a, 0, sizeof(a));
            a.q = a.k = a.v = a.o = a.dO = (const uint16_t *)(1 << 20);  // inputs here, outputs there, all strides 0
            a.lse_in = (const float *)(1 << 20);
            a.dq = a.dk = a.dv = (void *)((uintptr_t)1 << 40);
            const int grid = both_at_once(ctx, p, a);
            if (grid) {
                const int dkv = (int)p->pass[FLEXSP_PASS_BWD_DKV].direct.size(), dq = (int)p->pass[FLEXSP_PASS_BWD_DQ].direct.size();
                CHECK(dkv > 0 && dq > 0 && a.dkv_items == dkv && a.dq_wg >= dkv && a.dq_wg % ctx->num_xcd == 0 && grid == a.dq_wg + dq && dkv + dq <= 512);
                both++;
            }
            flexsp_plan_destroy(p);
        }
    }
    std::printf("%d lists, %d cut finer than listed, %d single launches, %d in halves\n", lists, finer, both, halves);
    CHECK(lists > 500 && finer > 100 && both > 200 && halves > 20);
    return 0;
}

// Which batches run in halves, either side of each line (256 compute units), that a plan which cuts no tile goes by it, and that a launch
// without a plan, which knows the rows of its tensors only, looks at the lengths of every batch that does and has workgroups for it.
static int check_halves(flexsp_ctx *ctx)
{
    const struct {
        std::vector<int> lens;
        int heads, D, causal;
        bool halves;
    } cases[] = {
        // tokens to a sequence, empty ones counted
        {{512}, 8, 128, 1, true}, {{511}, 8, 128, 1, false}, {{512}, 1, 64, 0, true}, {{511}, 1, 64, 0, false},
        {{1, 1700, 65}, 2, 128, 1, true}, {{0, 0, 1535}, 2, 128, 1, false}, {{0, 0, 1536}, 2, 128, 1, true},
        // one tile to a compute unit, whole tiles counted
        {{2048}, 8, 128, 0, true}, {{2049}, 8, 128, 0, false}, {{2048}, 8, 64, 0, true}, {{2049}, 8, 64, 0, false},
        {{1024}, 16, 128, 1, true}, {{1025}, 16, 128, 1, false}, {{960, 1024}, 8, 128, 0, true}, {{961, 1025}, 8, 128, 0, false},
        // more of them beside a long sequence: its length, all steps, all tiles
        {{2112}, 8, 128, 1, true}, {{2112}, 8, 128, 0, false}, {{2688}, 8, 128, 1, true}, {{2752}, 8, 128, 1, false}, {{1984, 832}, 6, 128, 1, false},
        {{1280, 1280}, 8, 128, 1, false}, {{2048, 960}, 7, 128, 1, true}, {{4096}, 5, 128, 0, false}, {{8192, 2048}, 2, 128, 0, false}, {{16384, 640}, 1, 128, 0, false}, {{9600, 2560, 2560, 2560}, 1, 128, 0, true},
        {{4032}, 8, 64, 1, true}, {{4096}, 8, 64, 1, false}, {{5120}, 7, 64, 1, true}, {{5120}, 8, 64, 1, false}, {{1984, 64}, 12, 64, 1, false},
        {{8192}, 2, 64, 0, true}, {{8192, 704}, 2, 64, 0, true}, {{20480}, 1, 64, 0, true}, {{20544}, 1, 64, 0, false}, {{32768, 16256}, 1, 64, 1, true},
    };
    int plans = 0;
    for (const auto &c : cases) {
        std::vector<int32_t> cu(1, 0);
        for (int s : c.lens) cu.push_back(cu.back() + s);
        const int B = (int)c.lens.size();
        flexsp_plan *p = nullptr;
        CHECK(flexsp_plan_create(ctx, cu.data(), B, c.heads, c.heads, c.D, c.causal, &p) == FLEXSP_OK);
        const HalvesCount n = halves_count(p);
        if (fwd_halves(c.D, n, 256) != c.halves) std::fprintf(stderr, "%d tokens, %d sequences, %d heads, D = %d, causal = %d\n", cu[B], B, c.heads, c.D, c.causal);
        CHECK(fwd_halves(c.D, n, 256) == c.halves);
        CHECK(p->halves == (c.halves && p->pass[FLEXSP_PASS_FWD].records == 0));
        plans += p->halves;
        if (c.halves)
            for (int64_t rows = cu[B]; rows < 100000; rows = rows * 3 / 2 + 1)
                CHECK(fwd_may_halve(rows, B, c.heads, 256) && fwd_halves_most(c.D, rows, B, c.heads, 256) >= n.tiles);
        flexsp_plan_destroy(p);
    }
    CHECK(plans >= 5);
    return 0;
}

// Whether a pass keeps the parts of one number of its cut tiles together or whole groups, either side of each line: sequences of the given
// lengths, `groups` groups (heads, or heads of keys) to each, a group walking `walked` heads, tiles as a forward's under a mask.
static int check_parts_kept(flexsp_ctx *ctx)
{
    const struct {
        std::vector<int> lens;
        int groups, walked, row_bytes;
        bool by_part;
    } cases[] = {
        {{20000}, 1, 1, 512, false}, {{20000}, 3, 1, 512, false}, {{20000}, 4, 1, 512, true}, {{20000}, 4, 1, 0, false},  // (0: no mask)
        {{7168}, 4, 1, 512, false}, {{7296}, 4, 1, 512, true}, {{14336}, 4, 1, 256, false}, {{14464}, 4, 1, 256, true},   // 3.5 MiB
        {{19381, 9000, 9000}, 1, 1, 512, false}, {{19381, 19381, 19381, 12000}, 1, 1, 512, false}, {{19381, 19381, 19381, 15000}, 1, 1, 512, true},
        {{30721}, 2, 4, 512, false}, {{12000}, 2, 4, 512, false}, {{30721}, 3, 4, 512, true}, {{8192}, 1, 8, 512, true}, {{3000}, 2, 8, 512, true},
    };
    for (const auto &c : cases) {
        std::vector<Work> work;
        std::vector<int64_t> cost;
        for (size_t b = 0; b < c.lens.size(); b++)
            for (int g = 0; g < c.groups; g++) {
                const int s = c.lens[b], tile = c.walked > 1 ? 64 : 128;
                cost.push_back(0);
                for (int t = 0; t * tile < s; t++) {
                    Work w;
                    std::memset(&w, 0, sizeof(w));
                    w.it.seq_len = s; w.it.tile = t; w.it.head = g;
                    w.cost = (cdiv(std::min(s, (t + 1) * tile), 64)) * c.walked;
                    w.group = (int32_t)cost.size() - 1;
                    cost.back() += w.cost;
                    work.push_back(w);
                }
            }
        HostPass hp;
        const size_t groups = cost.size(), tiles = work.size();
        const std::vector<int64_t> kept = split_long_items(work, cost, workgroups_of(ctx), 0, c.row_bytes, c.walked, hp);
        CHECK(work.size() > tiles && hp.records > 0);  // (some are cut)
        std::vector<int64_t> sum(kept.size(), 0);
        bool by_part = false;
        for (const Work &w : work) {
            CHECK(w.keep >= 0 && (size_t)w.keep < kept.size());
            sum[w.keep] += w.cost;
            if ((size_t)w.keep >= groups) {  // a number's list: of one group, of one number
                CHECK((w.it.parts & 0xffff) > 1 && (w.keep - (int)groups) % kMaxParts == w.it.parts >> 16);
                by_part = true;
            } else {
                CHECK(w.keep == w.group);
            }
        }
        CHECK(sum == kept);
        if (by_part != c.by_part) std::fprintf(stderr, "%d tokens first, %d groups of %d heads\n", c.lens[0], c.groups, c.walked);
        CHECK(by_part == c.by_part);
    }
    return 0;
}

// Which dK/dV passes have items of 128 keys, either side of each line (D = 64, 512 places): equal sequences.
static int check_wide_keys(flexsp_ctx *ctx)
{
    const struct {
        int n, len, hq, hkv, causal;
        bool wide;
    } cases[] = {
        {40, 740, 8, 8, 0, true}, {40, 704, 8, 8, 0, false}, {60, 512, 8, 8, 0, true}, {60, 384, 8, 8, 0, false}, {30, 1408, 8, 2, 1, true}, {30, 1280, 8, 2, 1, false},  // twelve steps to a walk
        {85, 200, 3, 3, 0, true}, {86, 200, 3, 3, 0, false}, {64, 200, 2, 2, 0, false}, {65, 200, 2, 2, 0, true},    // 256 and 512 items
        {100, 500, 1, 1, 1, true}, {100, 500, 4, 1, 1, false}, {100, 500, 4, 1, 0, true}, {100, 160, 8, 2, 0, false}, {100, 256, 8, 2, 0, true},
        {4, 900, 2, 2, 0, false}, {1, 6000, 1, 1, 1, false}, {1, 16384, 1, 1, 1, false}, {1, 32768, 1, 1, 1, true},  // (both passes in one launch)
    };
    for (const auto &c : cases) {
        std::vector<int32_t> cu(1, 0);
        for (int i = 0; i < c.n; i++) cu.push_back(cu.back() + c.len);
        flexsp_plan *p = nullptr;
        for (int D = 64; D <= 128; D *= 2) {
            CHECK(flexsp_plan_create(ctx, cu.data(), c.n, c.hq, c.hkv, D, c.causal, &p) == FLEXSP_OK);
            if (p->wide != (c.wide && D == 64)) std::fprintf(stderr, "%d of %d tokens, %d heads on %d, D = %d, causal = %d\n", c.n, c.len, c.hq, c.hkv, D, c.causal);
            CHECK(p->wide == (c.wide && D == 64) && p->pass[FLEXSP_PASS_BWD_DKV].tile_rows == (p->wide ? kDkvWideBk : kDkvBk));
            if (p->wide) {
                AttnArgs a;
                std::memset(&a, 0, sizeof(a));
                CHECK(both_at_once(ctx, p, a) == 0 && bwd_per_cu(ctx, p, FLEXSP_PASS_BWD_DKV) == 2);
            }
            flexsp_plan_destroy(p);
        }
    }
    return 0;
}

// Where a forward runs three workgroups per compute unit: D = 64 and no item of more than half a workgroup's share.
static int check_fwd_per_cu(flexsp_ctx *ctx)
{
    const struct {
        int n, len, heads, causal, per_cu;
    } cases[] = {{128, 512, 8, 1, 3}, {32, 2048, 8, 0, 3}, {2, 16384, 8, 0, 3}, {16, 2048, 4, 0, 3}, {15, 2048, 4, 0, 2}, {16, 2048, 4, 1, 2}, {31, 2048, 4, 1, 3}};
    for (const auto &c : cases)
        for (int D = 64; D <= 128; D *= 2) {
            std::vector<int32_t> cu(1, 0);
            for (int i = 0; i < c.n; i++) cu.push_back(cu.back() + c.len);
            flexsp_plan *p = nullptr;
            CHECK(flexsp_plan_create(ctx, cu.data(), c.n, c.heads, c.heads, D, c.causal, &p) == FLEXSP_OK);
            const HostPass &f = p->pass[FLEXSP_PASS_FWD];
            if (fwd_per_cu(ctx, p) != (D == 64 ? c.per_cu : 2)) std::fprintf(stderr, "%d of %d tokens, %d heads: longest %ld of %ld steps\n", c.n, c.len, c.heads, (long)f.longest, (long)f.steps);
            CHECK(fwd_per_cu(ctx, p) == (D == 64 ? c.per_cu : 2));
            flexsp_plan_destroy(p);
        }
    return 0;
}

int main()
{
    flexsp_ctx *ctx = nullptr;
    CHECK(flexsp_ctx_create(&ctx, -1) == FLEXSP_OK);
    if (check_overlap(ctx) || check_direct_lists(ctx) || check_halves(ctx) || check_parts_kept(ctx) || check_wide_keys(ctx) || check_fwd_per_cu(ctx)) return 1;
    flexsp_ctx_destroy(ctx);
    std::puts("launch decisions: ok");
    return 0;
}
