"""The forward without a plan where more items than there are workgroups are found in the lengths, by the workgroups or by a kernel in front that lists them: against the plan's forward, bit
for bit, also where both cut long tiles into the same parts (where only the plan does, or there are not records enough for its parts, to
within the rounding of fp32 sums and of the bf16 store); up to and beyond as many sequences as are searched; wrong lengths; call after call."""
import numpy as np
import pytest

from paper_2412_01523_amd import workloads as wl

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2412_01523_amd import binding as fx
    c = fx.Context(0)
    yield c
    c.close()


#        lengths, rows beyond them, heads, key heads, D, causal, cut
CASES = {
    "one-sequence-cut": ([33000], 0, 2, 1, 128, True, True),
    "one-sequence-cut-d64": ([33001], 7, 2, 2, 64, True, True),
    "more-parts-than-records": ([36001], 0, 2, 2, 64, True, "other parts"),
    "fewer-parts-for-the-records": ([34501], 0, 2, 2, 64, True, "other parts"),
    "cut-beside-short-ones": ([9001, 1, 0, 128, 129, 127, 64, 65] * 2 + [300] * 150, 0, 3, 3, 128, True, True),
    "not-causal-cut": ([70, 4000, 0, 3969] + [500] * 150, 100, 1, 1, 128, False, True),
    "last-tile-of-one-step": ([128 * 9 + 1, 128 * 9, 128 * 9 + 64, 128 * 9 + 65] * 8, 0, 8, 2, 128, True, False),
    "heads-16": ([2000, 1000, 3, 700] * 2 + [90] * 20, 0, 16, 2, 64, True, "by the plan only"),
    "heads-12-not-causal": ([700, 0, 513, 512, 1] * 5, 0, 12, 4, 128, False, False),
    "heads-8-cut": ([4300] + [30] * 31, 0, 8, 4, 128, True, True),
    "heads-8-cut-d64": ([4100, 1] + [30] * 31, 3, 8, 2, 64, True, True),
    "heads-8-cut-listed": ([30] * 100 + [4300] + [30] * 100, 0, 8, 4, 128, True, True),
    "heads-8-cut-in-many-rows": ([4300] + [30] * 31, 31000, 8, 4, 128, True, True),
    "1792-items": ([130] * 100, 2872, 8, 2, 64, True, False),
    "1800-items": ([130] * 100, 2873, 8, 2, 64, True, False),
    "listed-not-causal": ([1, 700, 0, 129, 513] * 20, 3, 12, 3, 64, False, False),
    "listed-9-heads": ([260] * 80, 0, 9, 9, 128, True, False),
    "64-sequences": ([130, 128] * 32, 0, 8, 8, 128, True, False),
    "65-sequences": ([257] * 64 + [1], 0, 8, 8, 64, False, False),
    "256-sequences": ([i % 300 for i in range(256)], 5, 4, 2, 128, True, False),
    "300-sequences-16-heads": ([i % 300 for i in range(300)], 7, 16, 4, 64, True, False),
    "300-sequences-8-heads": ([i % 200 for i in range(300)], 0, 8, 8, 128, False, False),
    "257-sequences": ([i % 300 for i in range(257)], 5, 4, 2, 128, True, False),
}


@pytest.mark.parametrize("name", CASES)
def test_same_bits_as_with_a_plan(ctx, name):
    import torch
    from paper_2412_01523_amd import binding as fx
    lens, more, hq, hkv, D, causal, cut = CASES[name]
    print(f"static forward, items found in the lengths: {name}", flush=True)
    cu, T = wl.cu_seqlens(lens), sum(lens)
    rows = T + more
    q, k, v = (torch.full((rows, h, D), float("nan"), dtype=torch.bfloat16, device="cuda") for h in (hq, hkv, hkv))
    for tid, x in ((0, q), (1, k), (2, v)):
        x[:T] = to_dev(wl.normal_bf16(881, tid, (T, x.shape[1], D)))
    cud = torch.from_numpy(cu).cuda()
    want, want_lse = torch.empty((T, hq, D), dtype=torch.bfloat16, device="cuda"), torch.empty((hq, T), dtype=torch.float32, device="cuda")
    plan = fx.Plan(ctx, cu, hq, hkv, D, causal)
    assert (plan.items(fx.PASS_FWD)[0]["nparts"] > 1).any() == bool(cut)
    fx.flexsp_attn_varlen_fwd(ctx, plan, q[:T], k[:T], v[:T], cud, want, want_lse, causal=causal)
    torch.cuda.synchronize()
    plan.close()
    for _ in range(3):
        o = torch.full((rows, hq, D), 7.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, rows), 7.0, dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd_static(ctx, q, k, v, cud, o, lse, causal=causal)
        torch.cuda.synchronize()
        if isinstance(cut, str):
            a, b = o[:T].double(), want.double()
            assert float((a - b).abs().max()) <= 2.0 ** -7 * float(b.abs().max()) + 1e-6 and float((a - b).norm() / b.norm()) <= 1e-3
            assert float((lse[:, :T] - want_lse).abs().max()) <= 1e-5 * (1 + float(want_lse.abs().max()))
        else:
            assert torch.equal(o[:T].view(torch.int16), want.view(torch.int16))
            assert torch.equal(lse[:, :T].view(torch.int32), want_lse.view(torch.int32))
        assert bool((o[T:] == 7.0).all()) and bool((lse[:, T:] == 7.0).all())


# (a longest tile of 59 steps beside an even share of 34; unmasked, 58 beside 18 on fewer tiles than compute units)
@pytest.mark.parametrize("lens,hq,hkv,D,causal", [([3776, 507, 1386, 539], 16, 4, 128, True), ([3700] + [77] * 52, 6, 3, 128, False)])
def test_tiles_that_do_not_outlast_the_rest_stay_whole(ctx, lens, hq, hkv, D, causal):
    """The first sequence has the bits of a call of its own, which has too few items to be dealt and cuts nothing."""
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"static forward, whole tiles: {lens[0]} tokens beside {len(lens) - 1} sequences, {hq} heads", flush=True)
    T, n = sum(lens), lens[0]
    q, k, v = (to_dev(wl.normal_bf16(884, tid, (T, h, D))) for tid, h in ((0, hq), (1, hkv), (2, hkv)))
    outs = []
    for x in (lens, [n]):
        t = sum(x)
        o, lse = torch.empty((t, hq, D), dtype=torch.bfloat16, device="cuda"), torch.empty((hq, t), dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd_static(ctx, q[:t], k[:t], v[:t], torch.from_numpy(wl.cu_seqlens(x)).cuda(), o, lse, causal=causal)
        outs.append((o[:n], lse[:, :n].contiguous()))
    torch.cuda.synchronize()
    assert torch.equal(outs[0][0].view(torch.int16), outs[1][0].view(torch.int16)) and torch.equal(outs[0][1].view(torch.int32), outs[1][1].view(torch.int32))


@pytest.mark.parametrize("cu", [[1, 8000], [0, 9000, 8000], [0, 8000, 8000 + 4097], [0, -1, 8000], [0, 0, 0]])
def test_wrong_or_no_lengths_touch_nothing(ctx, cu):
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"static forward, wrong lengths: {cu}", flush=True)
    T, h = 12096, 8
    q, k, v = (to_dev(wl.normal_bf16(882, tid, (T, h, 128))) for tid in (0, 1, 2))
    o = torch.full((T, h, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((h, T), 7.0, dtype=torch.float32, device="cuda")
    for lens in (cu, [0, 12096], cu):  # (a good call between: tickets and arrivals are clear after either)
        o.fill_(7.0)
        lse.fill_(7.0)
        cud = torch.tensor(lens + [lens[-1]] * (8 - len(lens)), dtype=torch.int32).cuda()
        fx.flexsp_attn_varlen_fwd_static(ctx, q, k, v, cud, o, lse)
        torch.cuda.synchronize()
        good = lens is not cu
        assert bool((o == 7.0).all()) != good and bool((lse == 7.0).all()) != good
        assert not good or bool(torch.isfinite(lse).all())


@pytest.mark.parametrize("rows", [8192, 36000])  # (items found by the workgroups; listed in front)
def test_replayed_dealt_and_cut(ctx, rows):
    """One captured call whose batches are dealt whole, dealt with tiles cut, and small enough for neither, in turn: each replay starts from the
    counters that the one before left, and has the plan's bits."""
    import torch
    from paper_2412_01523_amd import binding as fx
    hq, hkv, D, B = 8, 4, 128, 32
    q, k, v = (to_dev(wl.normal_bf16(883, tid, (rows, h, D))) for tid, h in ((0, hq), (1, hkv), (2, hkv)))
    cud = torch.from_numpy(wl.cu_seqlens([128] * B)).cuda()
    o, lse = torch.empty((rows, hq, D), dtype=torch.bfloat16, device="cuda"), torch.empty((hq, rows), dtype=torch.float32, device="cuda")
    call = lambda: fx.flexsp_attn_varlen_fwd_static(ctx, q, k, v, cud, o, lse)  # noqa: E731
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call()
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call()
    whole, cut, short = [260] * 31 + [1], [4300] + [30] * 31, [64] * 32
    for lens in (whole, cut, cut, short, cut, whole, whole, cut):
        cu, T = wl.cu_seqlens(lens), sum(lens)
        print(f"static forward, captured: {lens[0]} tokens in the first of {B} sequences", flush=True)
        cud.copy_(torch.from_numpy(cu))
        o.fill_(7.0)
        lse.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        plan = fx.Plan(ctx, cu, hq, hkv, D)
        assert (plan.items(fx.PASS_FWD)[0]["nparts"] > 1).any() == (lens is cut)
        want, want_lse = torch.empty((T, hq, D), dtype=torch.bfloat16, device="cuda"), torch.empty((hq, T), dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd(ctx, plan, q[:T], k[:T], v[:T], cud, want, want_lse)
        torch.cuda.synchronize()
        plan.close()
        assert torch.equal(o[:T].view(torch.int16), want.view(torch.int16)) and torch.equal(lse[:, :T].view(torch.int32), want_lse.view(torch.int32))
        assert bool((o[T:] == 7.0).all()) and bool((lse[:, T:] == 7.0).all())
