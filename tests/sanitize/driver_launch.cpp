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

int main()
{
    flexsp_ctx *ctx = nullptr;
    CHECK(flexsp_ctx_create(&ctx, -1) == FLEXSP_OK);
    if (check_overlap(ctx)) return 1;
    flexsp_ctx_destroy(ctx);
    std::puts("launch decisions: ok");
    return 0;
}
