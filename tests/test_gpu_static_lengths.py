"""The forward without a plan finds its work on the device: every workgroup one item for itself where the batch fits the chip at once, dealt
items (test_gpu_static_search.py) or a list where it does not.  Same bits as the plan's forward around that line and at odd lengths, however many rows the tensors hold."""
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


def both(ctx, lens, hq, hkv, D, causal):
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"static forward: {len(lens)} sequences, {sum(lens)} tokens, {hq} heads on {hkv}, D={D}, causal={causal}", flush=True)
    cu, T = wl.cu_seqlens(lens), sum(lens)
    q, k, v = (to_dev(wl.normal_bf16(771, tid, (T, h, D))) for tid, h in ((0, hq), (1, hkv), (2, hkv)))
    cud = torch.from_numpy(cu).cuda()
    outs = []
    for planned in (True, False):
        o = torch.full((T, hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, T), float("nan"), dtype=torch.float32, device="cuda")
        if planned:
            with_plan = fx.Plan(ctx, cu, hq, hkv, D, causal)
            assert int(with_plan.items(fx.PASS_FWD)[0]["nparts"].max()) == 1
            fx.flexsp_attn_varlen_fwd(ctx, with_plan, q, k, v, cud, o, lse, causal=causal)
            torch.cuda.synchronize()
            with_plan.close()
        else:
            fx.flexsp_attn_varlen_fwd_static(ctx, q, k, v, cud, o, lse, causal=causal)
            torch.cuda.synchronize()
        outs.append((o.view(torch.int16), lse.view(torch.int32)))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


# (ceil(T / 128) + B) x heads is the bound the choice is made by: 512 items and one more sequence
@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 253, 254, 255, 256, 600])
@pytest.mark.parametrize("causal", [True, False])
def test_many_sequences(ctx, n, causal):
    both(ctx, [1 + (37 * i) % 130 if i % 5 else 0 for i in range(n - 1)] + [129], 2, 1, 64, causal)


# (lengths whose tiles the plan leaves whole: up to 31 steps of 64 keys, or less than an even share of the pass)
@pytest.mark.parametrize("lens,hq,hkv,D", [([1], 1, 1, 128), ([128], 16, 2, 128), ([1153, 1, 0, 640], 6, 3, 128), ([1900], 16, 2, 128),
                                           ([0, 0, 700, 0], 4, 4, 64), ([1000] * 70, 3, 1, 64), ([9000] * 9 + [4500], 7, 7, 64)])
def test_odd_shapes(ctx, lens, hq, hkv, D):
    both(ctx, lens, hq, hkv, D, True)


@pytest.mark.parametrize("T,B", [(1024, 3), (65536, 200), (4096, 2), (65536, 2), (200000, 100), (30000, 300)])  # (the third and fourth: batches that might run in halves; the last two: listed)
def test_wrong_lengths_compute_nothing(ctx, T, B):
    import torch
    from paper_2412_01523_amd import binding as fx
    good = [i * T // B for i in range(B + 1)]
    for at, value in ((0, 1), (B // 2, -1), (B // 2, T + 1), (B, T + 1), (B, 0)):
        cu = torch.tensor(good, dtype=torch.int32)
        cu[at] = value
        t = torch.zeros((T, 2, 64), dtype=torch.bfloat16, device="cuda")
        o, lse = torch.full_like(t, 7.0), torch.full((2, T), 7.0, dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd_static(ctx, t, t, t, cu.cuda(), o, lse)
        torch.cuda.synchronize()
        assert bool((o == 7.0).all()) and bool((lse == 7.0).all()), (at, value)


# Tensors with room for more tokens than the batch has, whose lengths alone say how the forward runs: in one launch that takes
# the batch either way, with items found one to a workgroup or dealt, and (the last ones) batches that are not for halves
@pytest.mark.parametrize("lens,hq,hkv,D,rows", [
    ([1000], 8, 8, 128, 1000), ([1000], 8, 8, 128, 1900), ([1000], 8, 8, 128, 4096), ([1000], 8, 2, 128, 9000), ([1900], 8, 8, 128, 4096),
    ([700, 0, 1301], 2, 1, 128, 8192), ([700, 0, 1301], 2, 2, 128, 40000), ([900, 450], 4, 4, 64, 4096), ([1500], 4, 2, 64, 17000),
    ([8400], 4, 2, 64, 17000), ([0, 0, 700], 4, 4, 64, 2048), ([300, 200], 4, 4, 128, 4096), ([64], 1, 1, 128, 640), ([511], 8, 8, 128, 1000), ([1], 16, 4, 64, 30000),
], ids=lambda x: str(x).replace(" ", ""))
@pytest.mark.parametrize("causal", [True, False])
def test_room_for_more_tokens_changes_nothing(ctx, lens, hq, hkv, D, rows, causal):
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"static forward: {lens} in {rows} rows, {hq} heads on {hkv}, D={D}, causal={causal}", flush=True)
    cu, T = wl.cu_seqlens(lens), sum(lens)
    q, k, v = (torch.full((rows, h, D), float("nan"), dtype=torch.bfloat16, device="cuda") for h in (hq, hkv, hkv))
    for tid, x in ((0, q), (1, k), (2, v)):
        x[:T] = to_dev(wl.normal_bf16(772, tid, (T, x.shape[1], D)))
    cud = torch.from_numpy(cu).cuda()
    want, want_lse = torch.empty((T, hq, D), dtype=torch.bfloat16, device="cuda"), torch.empty((hq, T), dtype=torch.float32, device="cuda")
    plan = fx.Plan(ctx, cu, hq, hkv, D, causal)
    if int(plan.items(fx.PASS_FWD)[0]["nparts"].max()) == 1:
        fx.flexsp_attn_varlen_fwd(ctx, plan, q[:T], k[:T], v[:T], cud, want, want_lse, causal=causal)
        torch.cuda.synchronize()
    else:
        assert T == 8400  # (cut by the plan; here for the second turn that its halves take)
        fx.flexsp_attn_varlen_fwd_static(ctx, q[:T], k[:T], v[:T], cud, want, want_lse, causal=causal)
    plan.close()
    for _ in range(2):
        o = torch.full((rows, hq, D), 7.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, rows), 7.0, dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd_static(ctx, q, k, v, cud, o, lse, causal=causal)
        torch.cuda.synchronize()
        assert torch.equal(o[:T].view(torch.int16), want.view(torch.int16)) and torch.equal(lse[:, :T].view(torch.int32), want_lse.view(torch.int32))
        assert bool((o[T:] == 7.0).all()) and bool((lse[:, T:] == 7.0).all())


@pytest.mark.parametrize("rows,hq,D", [(2000, 8, 128), (4096, 8, 128), (9000, 8, 128), (4096, 4, 64), (17000, 4, 64)])
def test_replayed_with_other_lengths(ctx, rows, hq, D):
    """One captured call, the lengths changed between the replays: each runs as its lengths say, with the plan's bits."""
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"static forward, captured: {rows} rows, {hq} heads, D={D}", flush=True)
    q, k, v = (to_dev(wl.normal_bf16(773, tid, (rows, hq, D))) for tid in (0, 1, 2))
    cud = torch.tensor([0, 300, 700], dtype=torch.int32).cuda()
    o, lse = torch.empty((rows, hq, D), dtype=torch.bfloat16, device="cuda"), torch.empty((hq, rows), dtype=torch.float32, device="cuda")
    call = lambda: fx.flexsp_attn_varlen_fwd_static(ctx, q, k, v, cud, o, lse)  # noqa: E731
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call()
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call()
    for lens in ([1000, 200], [300, 400], [0, 1900], [900, 900], [64, 1]):
        cu, T = wl.cu_seqlens(lens), sum(lens)
        cud.copy_(torch.from_numpy(cu))
        o.fill_(7.0)
        lse.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        plan = fx.Plan(ctx, cu, hq, hq, D)
        assert int(plan.items(fx.PASS_FWD)[0]["nparts"].max()) == 1
        want, want_lse = torch.empty((T, hq, D), dtype=torch.bfloat16, device="cuda"), torch.empty((hq, T), dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd(ctx, plan, q[:T], k[:T], v[:T], cud, want, want_lse)
        torch.cuda.synchronize()
        plan.close()
        assert torch.equal(o[:T].view(torch.int16), want.view(torch.int16)) and torch.equal(lse[:, :T], want_lse), lens
        assert bool((o[T:] == 7.0).all()) and bool((lse[:, T:] == 7.0).all()), lens
