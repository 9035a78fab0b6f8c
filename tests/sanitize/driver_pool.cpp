// The memory of plans, against a HIP runtime of a few lines with as much memory as a test gives it: what a plan takes from the context's pool,
// what is given back before an allocation is given up, and that a backward falls back to two passes.  csrc/flexsp_host.hip is part of this program.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>

namespace fake {
size_t limit = ~(size_t)0, used = 0;
int mallocs = 0, waits = 0;
std::map<void *, size_t> device;
std::set<void *> pending;  // events of kernels that have not finished
hipError_t alloc(void **p, size_t n)
{
    mallocs++;
    *p = nullptr;
    if (n + used > limit) return hipErrorOutOfMemory;
    *p = std::malloc(1);  // (nothing looks inside)
    device[*p] = n;
    used += n;
    return hipSuccess;
}
hipError_t release(void *p)
{
    used -= device.at(p);
    device.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t host_alloc(void **p, size_t n)
{
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t host_release(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t event(hipEvent_t *e)
{
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t drop(hipEvent_t e)
{
    pending.erase(e);
    std::free(e);
    return hipSuccess;
}
hipError_t wait(hipEvent_t e)
{
    waits += (int)pending.erase(e);
    return hipSuccess;
}
hipError_t record(hipEvent_t e, hipStream_t s)
{
    if (s) pending.insert(e);  // (the upload's stream is the null one here)
    return hipSuccess;
}
}  // namespace fake
#define hipMalloc(p, n) fake::alloc(p, n)
#define hipMemGetInfo(f, t) (*(f) = fake::limit > fake::used ? fake::limit - fake::used : 0, *(t) = fake::limit, hipSuccess)
#define hipFree(p) fake::release(p)
#define hipHostMalloc(p, n, f) fake::host_alloc(p, n)
#define hipHostFree(p) fake::host_release(p)
#define hipEventCreateWithFlags(e, f) fake::event(e)
#define hipEventDestroy(e) fake::drop(e)
#define hipEventQuery(e) (fake::pending.count(e) ? hipErrorNotReady : hipSuccess)
#define hipEventSynchronize(e) fake::wait(e)
#define hipEventRecord(e, s) fake::record(e, s)
#define hipStreamWaitEvent(s, e, f) hipSuccess
#define hipStreamSynchronize(s) hipSuccess
#define hipStreamDestroy(s) hipSuccess
#define hipDeviceSynchronize() hipSuccess
#define hipSetDevice(d) hipSuccess
#define hipGetLastError() hipSuccess
#define hipMemcpyAsync(d, s, n, k, st) hipSuccess

#include "flexsp_host.hip"

namespace flexsp {
int delta_launches = 0, dq_launches = 0, dkv_launches = 0;
hipError_t launch_pack(const void *, void *, int64_t, int, int, int, int, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_pack_many(int, const void *const *, void *const *, int64_t, const int32_t *, int, int, int, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_fwd(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_fwd_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dkv(const AttnArgs &, int, int, hipStream_t)
{
    dkv_launches++;
    return hipSuccess;
}
hipError_t launch_attn_bwd_dq(const AttnArgs &a, int, int, hipStream_t)
{
    (a.chain ? delta_launches : dq_launches)++;
    return hipSuccess;
}
hipError_t launch_attn_bwd_dkv_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_attn_bwd_dq_kvshard(const AttnArgs &, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_lse_merge(const uint16_t *, const float *, const uint16_t *, const float *, uint16_t *, float *, int64_t, int, int, int32_t, int32_t, int32_t,
                            int32_t, int32_t, int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_lse_merge_acc(float *, float *, const uint16_t *, const float *, uint16_t *, int64_t, int, int, int32_t, int32_t, int32_t, int32_t, int32_t,
                                int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t static_scratch_init(int) { return hipErrorUnknown; }
}  // namespace flexsp

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAILED: %s (line %d)\n", #c, __LINE__); return 1; } } while (0)

static flexsp_ctx *device_ctx()
{
    flexsp_ctx *ctx = nullptr;
    if (flexsp_ctx_create(&ctx, -1) != FLEXSP_OK) std::abort();
    ctx->device = 0;
    ctx->num_cu = 256;
    return ctx;
}

// `n` sequences of `len` tokens, eight heads
static flexsp_plan *make(flexsp_ctx *ctx, int n, int len, int *rc = nullptr)
{
    std::vector<int32_t> cu(1, 0);
    for (int i = 0; i < n; i++) cu.push_back(cu.back() + len);
    flexsp_plan *p = nullptr;
    const int r = flexsp_plan_create(ctx, cu.data(), n, 8, 8, 128, 1, &p);
    if (rc) *rc = r;
    return p;
}

static void use(flexsp_plan *p, intptr_t stream)
{
    p->used = true;
    p->last_stream = (hipStream_t)stream;
}

static int backward(flexsp_ctx *ctx, flexsp_plan *p)
{
    static char memory[64];
    const flexsp_tensor t{(void *)(((uintptr_t)memory + 15) & ~(uintptr_t)15), 8 * 128, 128};  // (nothing is launched)
    return flexsp_attn_varlen_bwd(ctx, p, t, t, t, t, t, (const float *)memory, nullptr, 0, 8, 0, 8, 1, 0.f, t, t, t, FLEXSP_BF16, (flexsp_stream)1);
}

int main()
{
    // a small plan does not take a large plan's memory, a somewhat smaller one does
    {
        flexsp_ctx *ctx = device_ctx();
        flexsp_plan *big = make(ctx, 32, 2048);
        CHECK(big && !big->chain.empty() && fake::used > (size_t)256 << 20);
        void *const dev = big->dev_base;
        flexsp_plan_destroy(big);
        flexsp_plan *small = make(ctx, 3, 300);
        CHECK(small && small->dev_base != dev && small->slab.dev_bytes < (size_t)64 << 20);
        flexsp_plan *next = make(ctx, 30, 2048);
        CHECK(next && next->dev_base == dev);
        flexsp_plan_destroy(next);
        flexsp_plan_destroy(small);
        // a slab of a few megabytes more is nobody's loss
        flexsp_plan *tiny = make(ctx, 1, 64);
        CHECK(tiny && tiny->dev_base != dev && fake::mallocs == 2);
        flexsp_plan_destroy(tiny);
        flexsp_ctx_destroy(ctx);
        CHECK(fake::used == 0);
    }
    // memory is short: what the pool holds is given back, first what has finished, then what has not, and the plan still runs in one pass
    {
        flexsp_ctx *ctx = device_ctx();
        flexsp_plan *a = make(ctx, 8, 2048), *b = make(ctx, 8, 2048), *c = make(ctx, 8, 2048);
        CHECK(a && b && c && !a->chain.empty());
        const size_t each = a->slab.dev_bytes;
        CHECK(fake::used == 3 * each);
        use(a, 1);  // its kernels run on
        flexsp_plan_destroy(a);
        flexsp_plan_destroy(b);
        flexsp_plan_destroy(c);
        CHECK(ctx->slabs.size() == 3 && fake::pending.size() == 1);
        fake::limit = 4 * each + each / 2;
        flexsp_plan *d = make(ctx, 24, 2048);  // about three times as much
        CHECK(d && !d->chain.empty() && ctx->slabs.size() == 1 && fake::waits == 0 && fake::pending.size() == 1);
        CHECK(backward(ctx, d) == FLEXSP_OK && flexsp::delta_launches == 1 && flexsp::dkv_launches == 1 && flexsp::dq_launches == 0);
        flexsp_plan_destroy(d);
        flexsp_plan *e = make(ctx, 32, 2048);  // four times: also the one that is in use, behind its kernels
        CHECK(e && !e->chain.empty() && ctx->slabs.empty() && fake::waits == 2 && fake::pending.empty());
        CHECK(ctx->slabs_owned == 1 && ctx->slab_bytes == e->slab.dev_bytes && fake::used == ctx->slab_bytes);
        flexsp_plan_destroy(e);
        flexsp_ctx_destroy(ctx);
        CHECK(fake::used == 0);
    }
    // not enough for one pass, with nothing in the pool: two passes, which need less; not enough for these: an error, and nothing held
    {
        flexsp_ctx *ctx = device_ctx();
        fake::limit = (size_t)100 << 20;
        flexsp_plan *p = make(ctx, 32, 2048);
        CHECK(p && p->chain.empty() && p->dq[FLEXSP_PASS_BWD_DQ].items);
        flexsp::delta_launches = flexsp::dkv_launches = 0;
        CHECK(backward(ctx, p) == FLEXSP_OK && flexsp::delta_launches == 0 && flexsp::dkv_launches == 1 && flexsp::dq_launches == 1);
        // (the next one does not give the pool's back in vain: it takes it)
        void *const dev = p->dev_base;
        flexsp_plan_destroy(p);
        fake::pending.clear();
        p = make(ctx, 32, 2048);
        CHECK(p && p->chain.empty() && p->dev_base == dev && ctx->slabs_owned == 1);
        flexsp_plan_destroy(p);
        flexsp_ctx_destroy(ctx);
        ctx = device_ctx();
        fake::limit = (size_t)1 << 20;
        int rc = 0;
        CHECK(!make(ctx, 32, 2048, &rc) && rc == FLEXSP_OUT_OF_MEMORY && fake::used == 0 && ctx->slabs_owned == 0 && ctx->slab_bytes == 0);
        fake::limit = ~(size_t)0;
        p = make(ctx, 32, 2048);
        CHECK(p && !p->chain.empty());
        flexsp_plan_destroy(p);
        flexsp_ctx_destroy(ctx);
    }
    // 4 GiB of rows are the most: 131 072 tiles of 64 rows and heads
    {
        flexsp_ctx *ctx = device_ctx();
        flexsp_plan *p = make(ctx, 512, 2048);
        CHECK(p && p->chain_tiles == kChainMostTiles && !p->chain.empty());
        flexsp_plan_destroy(p);
        p = make(ctx, 520, 2048);
        CHECK(p && p->chain.empty());
        flexsp_plan_destroy(p);
        flexsp_ctx_destroy(ctx);
    }
    CHECK(fake::used == 0 && fake::device.empty());
    std::printf("plan memory: ok\n");
    return 0;
}
