"""The ways a backward is launched, each named by what the library's own launch counts say and held against the CPU fp64 oracle:
both passes in one launch, two launches of one workgroup per item, two launches that deal their items."""
import numpy as np
import pytest

import oracle
from paper_2412_01523_amd import workloads as wl

from gpu_util import bf16_f64, check_against_budget, to_bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2412_01523_amd import binding as fx
    c = fx.Context(0)
    yield c
    c.close()


def launches(ctx, call):
    """(dK/dV launches, dQ launches) of what `call` does."""
    ctx.profile_start(16)
    call()
    p = ctx.profile_stop()
    assert p["dropped"] == 0
    return p["bwd_dkv"][1], p["bwd_dq"][1]


def inputs(seed, Tq, Tk, hq, hkv, D):
    q, g = (wl.normal_bf16(seed, tid, (Tq, hq, D)) for tid in (wl.TID_Q, wl.TID_DO))
    k, v = (wl.normal_bf16(seed, tid, (Tk, hkv, D)) for tid in (wl.TID_K, wl.TID_V))
    return q, k, v, g


# few items, and more than are resident at once
@pytest.mark.parametrize("lens,hq,hkv,D,causal,one", [
    ([300, 70], 2, 2, 128, True, True), ([513, 1, 130], 4, 2, 64, False, True), ([130, 1, 64, 257] * 20, 8, 4, 128, True, False),
])
def test_gradients_over_spent_inputs(ctx, lens, hq, hkv, D, causal, one):
    """dq over o, dk and dv over k and v: the two passes then run one after the other, whatever the size."""
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"overlap: {len(lens)} sequences, {hq} heads on {hkv}, D={D}, causal={causal}", flush=True)
    cu = wl.cu_seqlens(lens)
    T = int(cu[-1])
    q, k, v, g = inputs(921, T, T, hq, hkv, D)
    o, _, dq, dk, dv = oracle.attn_fwd_bwd(q, k, v, g, cu, causal)
    ref = {"O": o, "dQ": dq, "dK": dk, "dV": dv}
    plan = fx.Plan(ctx, cu, hq, hkv, D, causal)
    cud = torch.from_numpy(cu).cuda()

    def run(over):
        qd, kd, vd, gd = (to_dev(x) for x in (q, k, v, g))
        od, lse = torch.empty_like(qd), torch.empty((hq, T), dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd(ctx, plan, qd, kd, vd, cud, od, lse, causal=causal)
        out = {"O": bf16_f64(to_bits(od))}
        dqd, dkd, dvd = (od, kd, vd) if over else (torch.empty_like(x) for x in (od, kd, vd))
        n = launches(ctx, lambda: fx.flexsp_attn_varlen_bwd(ctx, plan, qd, kd, vd, od, gd, lse, cud, dqd, dkd, dvd, causal=causal))
        out.update(dQ=bf16_f64(to_bits(dqd)), dK=bf16_f64(to_bits(dkd)), dV=bf16_f64(to_bits(dvd)))
        return n, out

    for over in (False, True):
        n, out = run(over)
        assert n == ((1, 0) if one and not over else (1, 1))
        check_against_budget(f"over={over}", out, ref, q, k, v, g, cu, causal, None, False)
    plan.close()


# Short sequences beside the ones a case is about decide the route: with 4 heads on 2, `fillers` of at most 60 rows make
# 4 x fillers items of the dQ pass and 2 x fillers of the dK/dV pass, and up to 512 items (two per compute unit) are resident at once.
ROUTES = {"one launch": 0, "two launches, an item each": 70, "two launches, dealt": 300}


def check_route(ctx, plan, route, call):
    """The call is launched the way `route` says."""
    from paper_2412_01523_amd import binding as fx
    n = launches(ctx, call)
    assert n == ((1, 0) if route == "one launch" else (1, 1)), (route, n)
    items = [len(plan.items(which)[0]) for which in (fx.PASS_BWD_DKV, fx.PASS_BWD_DQ)]
    dealt = [i > 2 * ctx.num_cu for i in items]
    assert dealt == [route.startswith("two launches, dealt")] * 2, (route, items)


def filler(n, seed):
    return [int(x) for x in np.random.default_rng(seed).integers(1, 61, size=n)]


# (with D = 64 three workgroups share a compute unit where no item is more than half of a workgroup's share)
@pytest.mark.parametrize("D,causal,route", [(D, causal, route) for D in (128, 64) for causal in (True, False) for route in ROUTES] +
                         [(64, True, "two launches, dealt to three per unit")])
def test_shard_backward(ctx, D, causal, route):
    """One key shard, grouped heads: query tiles long enough to be cut, ragged ends on both sides, a sequence without keys, keys
    without queries, keys that nobody sees, rows that see none; bf16 and fp32 gradients, and fp32 added to what is there."""
    import torch
    from paper_2412_01523_amd import binding as fx
    hq, hkv, n = 4, 2, ROUTES.get(route, 600)
    three = route not in ROUTES
    lq = [130, 64, 0, 77, 200] + filler(n, 1)
    lk = [3001, 0, 50, 129, 100] + filler(n, 2)
    shift = [2900, 0, 0, -64, -90] + [int(x) for x in np.random.default_rng(3).integers(-20, 60, size=n)]
    if three:  # short ones only
        lq, lk, shift = lq[2:4] + lq[5:], lk[2:4] + lk[5:], shift[2:4] + shift[5:]
    print(f"shard backward: {route}, D={D}, causal={causal}", flush=True)
    cu_q, cu_k = wl.cu_seqlens(lq), wl.cu_seqlens(lk)
    q, k, v, g = inputs(923, sum(lq), sum(lk), hq, hkv, D)
    O, LSE = oracle.attn_fwd_kvshard(q, k, v, cu_q, cu_k, shift, causal)
    delta = np.einsum("thd,thd->ht", bf16_f64(g), O)
    ref = oracle.attn_bwd_kvshard(q, k, v, g, LSE, delta, cu_q, cu_k, shift, causal)
    unseen = int(cu_k[lq.index(0)])
    assert np.isneginf(LSE).any() and not ref[1][unseen:unseen + 50].any()
    plan = fx.ShardPlan(ctx, cu_q, cu_k, shift, hq, hkv, D, causal)
    if three:
        for which in (fx.PASS_BWD_DKV, fx.PASS_BWD_DQ):
            items = plan.items(which)[0]
            steps = items["step_end"] - items["step_begin"]
            assert 2 * steps.max() * 2 * ctx.num_cu <= steps.sum()
    elif n:
        assert (plan.items(fx.PASS_BWD_DQ)[0]["nparts"] > 1).any()
    qd, kd, vd, gd = (to_dev(x) for x in (q, k, v, g))
    od = to_dev(wl.f32_to_bf16_bits(O.astype(np.float32)))
    lse = torch.from_numpy(LSE.astype(np.float32)).cuda()
    shapes = [(sum(lq), hq, D), (sum(lk), hkv, D), (sum(lk), hkv, D)]
    gen = torch.Generator(device="cuda").manual_seed(924)
    for mode in ("bf16", "fp32", "accumulate"):
        dtype = torch.bfloat16 if mode == "bf16" else torch.float32
        before = [torch.randn(s, generator=gen, device="cuda") if mode == "accumulate" else torch.zeros(s, device="cuda") for s in shapes]
        runs = []
        for _ in range(2):
            out = [b.clone() if mode == "accumulate" else torch.full(s, float("nan"), dtype=dtype, device="cuda")
                   for b, s in zip(before, shapes)]
            check_route(ctx, plan, route, lambda: fx.flexsp_attn_varlen_bwd_kvshard(
                ctx, plan, qd, kd, vd, od, gd, lse, *out, causal=causal, accumulate=mode == "accumulate"))
            runs.append(out)
        for name, a, b, old, want in zip(("dQ", "dK", "dV"), *runs, before, ref):
            assert torch.equal(a, b), f"{mode} {name} is not reproducible"
            got = a.double().cpu().numpy() - old.double().cpu().numpy()
            assert np.isfinite(got).all(), f"{mode} {name}: non-finite values"
            # as for the other shard cases: 2e-2, or 5e-3 of the largest value where few keys are seen by many rows; a bf16
            # gradient's final rounding, 2^-8 of its value, and an fp32 sum's, 2^-24 of it, come on top
            tol = max(2e-2, 5e-3 * np.abs(want).max()) + np.abs(want) * (2.0 ** -8 if mode == "bf16" else 0) + \
                (np.abs(want) + np.abs(old.cpu().numpy())) * 2.0 ** -24
            worst = np.abs(got - want).max()
            assert (np.abs(got - want) <= tol).all(), f"{mode} {name}: {worst:.2e}"
            rel = np.sqrt(((got - want) ** 2).sum() / (want ** 2).sum())
            assert rel <= 5e-3, f"{mode} {name}: {rel:.2e}"
    plan.close()


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("D,causal", [(128, True), (64, True), (128, False), (64, False)])
def test_backward_of_head_subsets(ctx, D, causal, route):
    """Heads 4 .. 7 on key heads 1 .. 2 of wider tensors, written between guard bytes: tile edges, ragged and empty sequences, a
    sequence whose tiles are cut; the other heads and the guards keep what they hold."""
    import torch
    from paper_2412_01523_amd import binding as fx
    from test_gpu_invariants import Guarded
    hq, hkv, all_q, all_kv, n = 4, 2, 9, 4, ROUTES[route]
    lens = ([1, 128, 0, 129, 65, 640] if n == 0 else [1, 128, 0, 129, 65, 2100]) + filler(n, 4)
    print(f"head subset: {route}, D={D}, causal={causal}", flush=True)
    cu = wl.cu_seqlens(lens)
    T = int(cu[-1])
    q, k, v, g = inputs(925, T, T, all_q, all_kv, D)
    mine_q, mine_kv = slice(4, 4 + hq), slice(1, 1 + hkv)
    dense = [np.ascontiguousarray(x[:, s]) for x, s in ((q, mine_q), (k, mine_kv), (v, mine_kv), (g, mine_q))]
    O, LSE, dQ, dK, dV = oracle.attn_fwd_bwd(*dense, cu, causal)
    ref = {"O": O, "dQ": dQ, "dK": dK, "dV": dV}
    plan = fx.Plan(ctx, cu, hq, hkv, D, causal)
    if n:
        assert (plan.items(fx.PASS_BWD_DQ)[0]["nparts"] > 1).any()
    qd, kd, vd, gd = (to_dev(x) for x in (q, k, v, g))
    cud = torch.from_numpy(cu).cuda()
    od = torch.zeros((T, all_q, D), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((hq, T), dtype=torch.float32, device="cuda")
    heads = dict(head_begin=4, head_count=hq, kv_head_begin=1, kv_head_count=hkv)
    fx.flexsp_attn_varlen_fwd(ctx, plan, qd, kd, vd, cud, od, lse, causal=causal, **heads)
    assert np.abs(lse.cpu().numpy() - LSE).max() < 1e-3
    for f32 in (True, False):
        bufs = [Guarded((T, h, D), torch.float32 if f32 else torch.bfloat16) for h in (all_q, all_kv, all_kv)]
        for b in bufs:
            b.t.fill_(7.0)
        check_route(ctx, plan, route, lambda: fx.flexsp_attn_varlen_bwd(
            ctx, plan, qd, kd, vd, od, gd, lse, cud, *(b.t for b in bufs), causal=causal, **heads))
        out = {"O": od[:, mine_q].double().cpu().numpy()}
        for name, b, s in zip(("dQ", "dK", "dV"), bufs, (mine_q, mine_kv, mine_kv)):
            assert b.guards_intact(), name
            out[name] = b.t[:, s].double().cpu().numpy()
            assert (b.t[:, :s.start] == 7).all() and (b.t[:, s.stop:] == 7).all(), name
        check_against_budget(f"{route} f32={f32}", out, ref, *dense, cu, causal, None, f32)
    plan.close()
