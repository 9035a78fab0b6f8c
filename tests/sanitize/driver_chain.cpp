// The list of a backward in one pass, looked at from inside (csrc/flexsp_host.hip is part of this program): every key tile once, what an
// item waits for in front of it, bundles, shared rows apart, and either side of the line.  Host-only contexts, launchers that fail.
#include <cstdio>
#include <map>
#include <random>
#include <set>
#include <tuple>

#include "flexsp_host.hip"

namespace flexsp {
hipError_t launch_pack(const void *, void *, int64_t, int, int, int, int, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_pack_many(int, const void *const *, void *const *, int64_t, const int32_t *, int, int, int, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_fwd(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_fwd_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dkv(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dq(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dkv_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dq_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_lse_merge(const uint16_t *, const float *, const uint16_t *, const float *, uint16_t *, float *, int64_t, int, int, int32_t, int32_t, int32_t,
                            int32_t, int32_t, int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_lse_merge_acc(float *, float *, const uint16_t *, const float *, uint16_t *, int64_t, int, int, int32_t, int32_t, int32_t, int32_t, int32_t,
                                int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t static_scratch_init(int) { return hipErrorUnknown; }
}  // namespace flexsp

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAILED: %s (line %d)\n", #c, __LINE__); return 1; } } while (0)

// The two passes' lists of a plan that runs in one: made when they are asked for, and then what they would have been at once.
static int check_two_passes(flexsp_plan *p, int nq, int n_wg)
{
    for (int pass : {FLEXSP_PASS_BWD_DKV, FLEXSP_PASS_BWD_DQ}) CHECK(p->pass[pass].items.empty());
    CHECK(flexsp_plan_tile_rows(p, FLEXSP_PASS_BWD_DKV) == kDkvBk && flexsp_plan_tile_rows(p, FLEXSP_PASS_BWD_DQ) == kDqBq);
    for (int pass : {FLEXSP_PASS_BWD_DQ, FLEXSP_PASS_BWD_DKV}) {
        HostPass want;
        if (pass == FLEXSP_PASS_BWD_DKV)
            build_pass(p->cu, p->B, p->Hkv, p->Hq / p->Hkv, kDkvBk, kDkvBq, p->causal != 0, true, p->D, nq, n_wg, want);
        else
            build_pass(p->cu, p->B, p->Hq, 1, kDqBq, kDqBk, p->causal != 0, false, p->D, nq, n_wg, want);
        CHECK(flexsp_plan_num_items(p, pass) == (int64_t)want.items.size());
        std::vector<flexsp_item> got(want.items.size());
        int64_t offsets[kMaxQueues + 1];
        CHECK(flexsp_plan_get_items(p, pass, got.data(), (int64_t)got.size(), offsets) == FLEXSP_OK);
        CHECK(std::memcmp(got.data(), want.items.data(), got.size() * sizeof(flexsp_item)) == 0);
        for (int x = 0; x <= nq; x++) CHECK(offsets[x] == want.offsets[x]);
        CHECK(flexsp_plan_tile_rows(p, pass) == want.tile_rows);
    }
    return 0;
}

static int check_list(const flexsp_plan *p)
{
    const int G = p->Hq / p->Hkv;
    // bundles: all of the list, none empty
    CHECK(p->chain_bundles.front() == 0 && p->chain_bundles.back() == (int32_t)p->chain.size());
    std::vector<int32_t> bundle_of(p->chain.size());
    for (size_t b = 0; b + 1 < p->chain_bundles.size(); b++) {
        CHECK(p->chain_bundles[b] < p->chain_bundles[b + 1]);
        for (int32_t i = p->chain_bundles[b]; i < p->chain_bundles[b + 1]; i++) bundle_of[i] = (int32_t)b;
    }
    std::map<std::tuple<int, int, int>, int> at;  // (sequence, head, key tile) -> place
    for (size_t i = 0; i < p->chain.size(); i++) {
        const flexsp_item &it = p->chain[i];
        CHECK(at.emplace(std::make_tuple(it.seq_start, it.head, it.tile), (int)i).second);
    }
    std::set<std::pair<int64_t, int64_t>> kept;  // query tiles that are added to, of a sequence: disjoint ranges
    size_t items = 0;
    for (int b = 0; b < p->B; b++) {
        const int s = p->cu[b + 1] - p->cu[b], nt = (s + 63) / 64, nb = (s + 127) / 128;
        for (int g = 0; g < p->Hkv; g++)
            for (int t = 0; t < nb; t++) {
                const auto f = at.find(std::make_tuple(p->cu[b], g, t));
                CHECK(f != at.end());
                items++;
                const int i = f->second;
                const flexsp_item &it = p->chain[i];
                CHECK(it.seq_len == s && it.step_end == (nt - (p->causal ? 2 * t : 0)) * G && it.step_begin <= t);
                const int lead = at.at(std::make_tuple(p->cu[b], g, it.step_begin));
                CHECK(bundle_of[lead] == bundle_of[i] && lead <= i);
                if (t) {
                    const int before = at.at(std::make_tuple(p->cu[b], g, t - 1));
                    CHECK(before < i);  // what it waits for
                    CHECK((p->chain[before].parts != 0) == (bundle_of[before] != bundle_of[i]));
                    CHECK((it.step_begin == t) == (bundle_of[before] != bundle_of[i]));
                }
                if (t == nb - 1) CHECK(it.parts == 0);
                if (nb > 1) kept.emplace(it.slot, it.slot + nt);
            }
    }
    CHECK(items == p->chain.size());
    int64_t end = 0;
    for (const auto &k : kept) {
        CHECK(k.first >= end);
        end = k.second;
    }
    CHECK(end * p->Hq <= p->chain_tiles && p->chain_tiles <= kChainMostTiles);
    return 0;
}

int main()
{
    flexsp_ctx *ctx = nullptr;
    CHECK(flexsp_ctx_create(&ctx, -1) == FLEXSP_OK);
    std::mt19937 rng(7);
    int taken = 0;
    for (int n = 0; n < 200; n++) {
        const int hkv = 1 << (rng() % 4), hq = hkv << (rng() % 3), causal = rng() % 4 != 0, B = 1 + rng() % 40, most = 1 << (6 + rng() % 9);
        std::vector<int32_t> cu(1, 0);
        for (int b = 0; b < B; b++) cu.push_back(cu.back() + (int32_t)(rng() % 5 ? rng() % most : rng() % 3 * 64));
        flexsp_plan *p = nullptr;
        CHECK(flexsp_plan_create(ctx, cu.data(), B, hq, hkv, 128, causal, &p) == FLEXSP_OK);
        if (!p->chain.empty()) {
            taken++;
            if (check_list(p) || check_two_passes(p, ctx->num_xcd, workgroups_of(ctx))) return 1;
        }
        flexsp_plan_destroy(p);
    }
    CHECK(taken >= 20 && taken < 200);
    // the line (256 compute units): sequences of one length
    const struct {
        int n, len, hq, hkv, causal, D, chain;
    } cases[] = {
        {1, 131072, 8, 8, 1, 128, 1}, {1, 131072, 8, 8, 1, 64, 0}, {1, 131072, 3, 3, 1, 128, 0}, {16, 4096, 8, 8, 1, 128, 1}, {192, 256, 8, 8, 1, 128, 1},
        {300, 128, 8, 8, 1, 128, 0},   // two steps an item
        {32, 1024, 1, 1, 1, 128, 0}, {64, 1024, 1, 1, 1, 128, 1},  // 256 and 512 items
        {64, 768, 8, 8, 0, 128, 1}, {64, 704, 8, 8, 0, 128, 0},    // twelve steps an item, eleven, unmasked
        {8, 1024, 8, 8, 1, 128, 1}, {4, 2048, 8, 8, 1, 128, 1}, {2, 4096, 8, 8, 1, 128, 1},  // shares of 18, 34 and 66 steps, walks of 16, 32 and 64
        {1, 8192, 8, 8, 1, 128, 1}, {1, 8064, 8, 8, 1, 128, 0},   // 512 items and 504
        {32, 2048, 8, 8, 0, 128, 1}, {13, 1500, 8, 8, 0, 128, 0}, {41, 1600, 4, 4, 0, 128, 0},  // as many bundles for each die, or one more for some
        {5, 8192, 16, 4, 1, 128, 1}, {4, 8192, 16, 4, 1, 128, 0},  // 0.39 and 0.49 of a share: several heads to a key head
    };
    for (const auto &c : cases) {
        std::vector<int32_t> cu(1, 0);
        for (int i = 0; i < c.n; i++) cu.push_back(cu.back() + c.len);
        flexsp_plan *p = nullptr;
        CHECK(flexsp_plan_create(ctx, cu.data(), c.n, c.hq, c.hkv, c.D, c.causal, &p) == FLEXSP_OK);
        if (p->chain.empty() == (c.chain != 0)) std::fprintf(stderr, "%d of %d tokens, %d heads on %d, causal = %d, D = %d\n", c.n, c.len, c.hq, c.hkv, c.causal, c.D);
        CHECK(p->chain.empty() != (c.chain != 0));
        if (c.chain && check_list(p)) return 1;
        flexsp_plan_destroy(p);
    }
    flexsp_ctx_destroy(ctx);
    std::printf("chain lists: ok (%d of 200)\n", taken);
    return 0;
}
