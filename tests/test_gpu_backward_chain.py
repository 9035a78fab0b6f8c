"""The backward in one pass over the key tiles: against the CPU fp64 oracle at the edges of its tiles and bundles, both gradient modes, in
place, in a graph, and two of them at once."""
import numpy as np
import pytest

import oracle
from paper_2412_01523_amd import workloads as wl

from gpu_util import bf16_f64, check_against_budget, to_bits, to_dev
from test_gpu_backward_routes import inputs

pytestmark = pytest.mark.gpu

# sequences around the edges of query tiles (64), key tiles (128) and bundles (32 key tiles: 4 096 tokens), empty and one-token ones;
# one of several bundles beside short ones; grouped heads; without a mask
CASES = {
    "edges": ([4097, 1, 64, 65, 127, 0, 128, 129, 191, 255, 256, 257, 640, 4224, 2048] + [896] * 12, 8, 8, True),
    "short": ([130, 257, 383, 511, 300, 256] * 12, 8, 8, True),
    "grouped": ([900, 77, 1009, 128, 600, 881, 700, 870, 1, 936, 1000, 955, 640, 1024, 1, 961, 897] + [800] * 14, 16, 8, True),
    "unmasked": ([769, 1000, 833, 900, 1024, 961, 800, 895, 4100, 1025, 950] + [896] * 8, 8, 8, False),
}


def batch(name, seed=931, cases=CASES):
    lens, hq, hkv, causal = cases[name]
    T = sum(lens)
    return wl.cu_seqlens(lens), hq, hkv, causal, inputs(seed, T, T, hq, hkv, 128)


PLANS = []  # closed in front of their context, also those of a test that failed


class Backward:
    """A batch on the GPU, forward done; run() is its backward."""

    def __init__(self, ctx, name, seed=931, cases=CASES):
        import torch
        from paper_2412_01523_amd import binding as fx
        self.ctx, self.fx = ctx, fx
        self.cu, self.hq, self.hkv, self.causal, bits = batch(name, seed, cases)
        self.bits = bits
        self.q, self.k, self.v, self.g = (to_dev(x) for x in bits)
        self.cud = torch.from_numpy(self.cu).cuda()
        self.plan = fx.Plan(ctx, self.cu, self.hq, self.hkv, 128, self.causal)
        PLANS.append(self.plan)
        self.o, self.lse = torch.empty_like(self.q), torch.empty((self.hq, int(self.cu[-1])), dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd(ctx, self.plan, self.q, self.k, self.v, self.cud, self.o, self.lse, causal=self.causal)
        torch.cuda.synchronize()

    def outputs(self, dtype):
        import torch
        return [torch.full(x.shape, float("nan"), dtype=dtype, device="cuda") for x in (self.q, self.k, self.v)]

    def run(self, out, **kw):
        self.fx.flexsp_attn_varlen_bwd(self.ctx, self.plan, self.q, self.k, self.v, self.o, self.g, self.lse, self.cud, *out, causal=self.causal, **kw)
        return out


@pytest.fixture(scope="module")
def ctx():
    from paper_2412_01523_amd import binding as fx
    c = fx.Context(0)
    yield c
    while PLANS:
        PLANS.pop().close()
    c.close()


@pytest.mark.parametrize("name", CASES)
def test_against_the_oracle(ctx, name):
    import torch
    print(f"chain: {name}", flush=True)
    b = Backward(ctx, name)
    o, _, dq, dk, dv = oracle.attn_fwd_bwd(*b.bits, b.cu, b.causal)
    ref = {"O": o, "dQ": dq, "dK": dk, "dV": dv}
    f32 = b.outputs(torch.float32)
    ctx.profile_start(16)
    b.run(f32)
    p = ctx.profile_stop()
    assert [p[k][1] for k in ("bwd_delta", "bwd_dkv", "bwd_dq")] == [1, 1, 0]
    out = {"O": bf16_f64(to_bits(b.o))}
    out.update(zip(("dQ", "dK", "dV"), (x.double().cpu().numpy() for x in f32)))
    # (the budget that the roundings allow, element by element; the flat 2e-2 is a statement about other magnitudes: sums over a group's
    # heads and rows that see few keys pass it, by either backward)
    check_against_budget(f"{name} fp32", out, ref, *b.bits, b.cu, b.causal, None, True, stated=False)
    again = b.run(b.outputs(torch.float32))
    bf16 = b.run(b.outputs(torch.bfloat16))
    for n, x, y, z in zip(("dQ", "dK", "dV"), f32, again, bf16):
        assert torch.equal(x, y), f"{n} is not reproducible"
        assert torch.equal(x.to(torch.bfloat16), z), f"{n}: bf16 is not the fp32 result rounded once"
    # dq over o, dk and dv over k and v: read before they are overwritten
    over = b.run([b.o, b.k, b.v])
    for n, x, y in zip(("dQ", "dK", "dV"), bf16, over):
        assert torch.equal(x, y), f"{n} over an input"
    b.plan.close()


# sequences of several bundles (32 key tiles), heads that are no multiple of the compute dies: a head's next bundle is another die's, or comes
# back to the die that had the one before the last
LONG = {"six heads": ([16384], 6, 6, True), "beside short ones": ([12417, 9001] + [700] * 20, 5, 5, True), "unmasked, long": ([16384], 4, 4, False),
        "grouped, long": ([8200, 8192, 8192, 8192, 8192, 4000, 5000, 6000], 8, 4, True)}


@pytest.mark.parametrize("name", [*CASES, *LONG])
def test_rows_handed_from_die_to_die(ctx, name):
    """Against the two-kernel backward (as one key shard), three times.  dQ is the same sum of the same terms in the same order, the keys': the
    same bits, and rows that were read before the bundle in front had added to them for the last time would miss up to 128 keys' terms.
    dK and dV are summed from the last query rows to the first here."""
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"chain, long: {name}", flush=True)
    b = Backward(ctx, name, 951, {**CASES, **LONG})
    lens = np.diff(b.cu)
    plan = fx.ShardPlan(ctx, b.cu, b.cu, [0] * len(lens), b.hq, b.hkv, 128, b.causal)
    PLANS.append(plan)
    assert (plan.items(fx.PASS_BWD_DQ)[0]["nparts"] <= 1).all()  # (a cut tile's sums are formed apart)
    ref = b.outputs(torch.float32)
    fx.flexsp_attn_varlen_bwd_kvshard(ctx, plan, b.q, b.k, b.v, b.o, b.g, b.lse, *ref, causal=b.causal)
    for _ in range(3):
        ctx.profile_start(16)
        out = b.run(b.outputs(torch.float32))
        p = ctx.profile_stop()
        assert [p[k][1] for k in ("bwd_delta", "bwd_dkv", "bwd_dq")] == [1, 1, 0]
        # (zeros of either sign are equal: masked keys add them)
        assert torch.equal(out[0], ref[0]), f"dQ: {(out[0] != ref[0]).any(2).sum().item()} rows differ"
        # the largest difference of two orders of n terms: a rounding of 2^-24 of the sum so far for each of them.  Sixteen terms to a matrix
        # instruction, counted one by one; sums so far are taken to be no larger than four times the largest sum of a head
        n = int(lens.max()) * (b.hq // b.hkv)
        for what, x, y in zip(("dK", "dV"), out[1:], ref[1:]):
            assert ((x - y).abs().amax((0, 2)) <= n * 2.0 ** -24 * 4 * y.abs().amax((0, 2))).all(), what
            rel = ((x - y).double().norm() / y.double().norm()).item()
            assert rel <= n ** 0.5 * 2.0 ** -24, f"{what}: {rel:.1e}"
    plan.close()
    b.plan.close()


# (sequences whose last tile of query rows is half a tile)
NONFINITE = {"one pass": ([800, 992, 416] * 20, 8, 8, True), "two": ([800, 992, 416] * 20, 1, 1, True)}


@pytest.mark.parametrize("name", NONFINITE)
def test_a_row_that_is_not_finite(ctx, name):
    """A row of k, v, q or dO with an infinity or a NaN: what shares no visible pair's block of 32 rows and 32 keys with it keeps its bits."""
    import torch
    print(f"not finite: {name}", flush=True)
    b = Backward(ctx, name, 961, NONFINITE)
    clean = b.run(b.outputs(torch.float32))
    ctx.profile_start(16)
    b.run(b.outputs(torch.float32))
    assert (ctx.profile_stop()["bwd_delta"][1] == 1) == (name == "one pass")
    end = int(b.cu[-1])
    everywhere = torch.ones(end, dtype=torch.bool, device="cuda")

    def but(first, stop):
        keep = everywhere.clone()
        keep[first:stop] = False
        return keep

    for seq, row in ((0, 100), (1, 205), (4, 430), (16, 991), (17, 37), (3, 799), (2, 0)):
        start, stop = int(b.cu[seq]), int(b.cu[seq + 1])
        first = start + row // 32 * 32
        last = min(first + 32, stop)
        for which, x in (("k", b.k), ("v", b.v), ("q", b.q), ("dO", b.g)):
            # rows of dQ that see a key of the block, keys that are seen from a row of it
            if which in "kv":
                keep = but(first, stop), but(first, last), but(first, last)
            else:
                keep = but(first, last), but(start, last), but(start, last)
            for value in (float("inf"), float("nan")):
                old = x[start + row].clone()
                x[start + row, :, 5:9] = value
                out = b.run(b.outputs(torch.float32))
                for n, got, want, rows in zip(("dQ", "dK", "dV"), out, clean, keep):
                    assert torch.equal(got[rows], want[rows]), f"{which}[{seq}, {row}] = {value}: {n}"
                if which == "dO" and row == 799 and value > 0:  # a last half tile: nothing but P times infinity, P > 0
                    assert (out[2][start:stop, :, 5:9] == value).all(), "dV"
                x[start + row] = old
    b.plan.close()


@pytest.mark.parametrize("name", ["edges", "grouped", "unmasked"])
@pytest.mark.parametrize("f32", [False, True])
def test_views_and_head_subsets(ctx, name, f32):
    """Some heads of wider tensors whose rows and heads lie apart, each tensor its own way: the dense tensors' bits, and nothing beside them."""
    import torch
    print(f"chain, views: {name}, f32={f32}", flush=True)
    b = Backward(ctx, name)
    T, dtype = int(b.cu[-1]), torch.float32 if f32 else torch.bfloat16
    ref = b.run(b.outputs(dtype))
    first_q, first_kv = 3, 1

    def wide(x, first, heads, d):  # rows of `heads` heads of d elements, the first 128 of each
        t = torch.full((T + 2, first + heads, d), 7.0, dtype=x.dtype, device="cuda")
        v = t[1:-1, :, :128]
        v[:, first:first + x.shape[1]] = x
        return t, v

    q, g, o = (wide(x, first_q, b.hq + n, d)[1] for x, n, d in ((b.q, 0, 136), (b.g, 2, 128), (b.o, 1, 192)))
    k, v = (wide(x, first_kv, b.hkv + n, d)[1] for x, n, d in ((b.k, 3, 144), (b.v, 0, 128)))
    outs = [wide(torch.full_like(x, 7.0), first, x.shape[1] + n, d)
            for x, first, n, d in zip(ref, (first_q, first_kv, first_kv), (1, 0, 2), (160, 128, 136))]
    ctx.profile_start(16)
    b.fx.flexsp_attn_varlen_bwd(ctx, b.plan, q, k, v, o, g, b.lse, b.cud, *(x for _, x in outs), causal=b.causal,
                                head_begin=first_q, head_count=b.hq, kv_head_begin=first_kv, kv_head_count=b.hkv)
    assert ctx.profile_stop()["bwd_delta"][1] == 1
    for n, (t, view), want, first in zip(("dQ", "dK", "dV"), outs, ref, (first_q, first_kv, first_kv)):
        mine = view[:, first:first + want.shape[1]]
        assert torch.equal(mine, want), n
        mine.fill_(7.0)
        assert (t == 7).all(), f"{n}: written beside"
    b.plan.close()


def test_replayed_from_a_graph(ctx):
    import torch
    b = Backward(ctx, "edges")
    ref = [x.clone() for x in b.run(b.outputs(torch.bfloat16))]
    torch.cuda.synchronize()
    out = b.outputs(torch.bfloat16)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        b.run(out, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    for rep in range(3):
        for t in out:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for x, y in zip(ref, out):
            assert torch.equal(x, y), f"replay {rep}"
        b.run(b.outputs(torch.bfloat16))  # the program's own eager work between replays
        torch.cuda.synchronize()
    b.plan.close()


def test_two_at_once(ctx):
    """Two plans on two streams: their workgroups take each other's compute units, and what either waits for is always running."""
    import torch
    pair = [Backward(ctx, "edges", 941), Backward(ctx, "short", 942)]
    refs = [[x.clone() for x in b.run(b.outputs(torch.bfloat16))] for b in pair]
    outs = [b.outputs(torch.bfloat16) for b in pair]
    streams = [torch.cuda.Stream() for _ in pair]
    torch.cuda.synchronize()
    for _ in range(10):
        for b, out, s in zip(pair, outs, streams):
            b.run(out, stream=s)
    torch.cuda.synchronize()
    for b, ref, out in zip(pair, refs, outs):
        assert all(torch.equal(x, y) for x, y in zip(ref, out))
        b.plan.close()


def test_plans_behind_a_full_pool():
    """A larger plan than any of those that fill the context's pool is kept like they were: the next one takes its memory over."""
    import torch
    from paper_2412_01523_amd import binding as fx
    ctx = fx.Context(0)
    few = [fx.Plan(ctx, wl.cu_seqlens([300]), 2, 2, 64, True) for _ in range(17)]
    for p in few:
        p.close()
    free = []
    for _ in range(3):
        p = fx.Plan(ctx, wl.cu_seqlens([2048] * 32), 8, 8, 128, True)  # 256 MB of dQ's rows, a quarter more as allocated
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
        p.close()
        free.append(torch.cuda.mem_get_info()[0])
    ctx.close()
    assert max(free) - min(free) < 160 << 20, free  # (one of the few, under 100 MB, is given back at first)
