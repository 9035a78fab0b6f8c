"""Launches of few items: one workgroup per item, both backward passes in one launch, tiles cut into short parts; and the
sizes around the lines where each of these ends: against the CPU fp64 oracle, twice."""
import numpy as np
import pytest

import oracle
from paper_2412_01523_amd import workloads as wl

from gpu_util import GpuAttn, check_against_budget

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2412_01523_amd import binding as fx
    c = fx.Context(0)
    yield c
    c.close()


def case_lengths(items, head_items):
    """`items` work items in every pass: sequences of at most 64 tokens with `head_items` heads each, one item per head."""
    n = items // head_items
    return [1 + (7 * i) % 5 for i in range(n - 1)] + [61]


def check(ctx, lens, hq, hkv, D, causal, grad_f32=True, stated=True):
    print(f"launch shape: {len(lens)} sequences, {hq} heads on {hkv}, D={D}, causal={causal}", flush=True)
    cu = wl.cu_seqlens(lens)
    T = int(cu[-1])
    q, dO = (wl.normal_bf16(911, tid, (T, hq, D)) for tid in (wl.TID_Q, wl.TID_DO))
    k, v = (wl.normal_bf16(911, tid, (T, hkv, D)) for tid in (wl.TID_K, wl.TID_V))
    o, lse, dq, dk, dv = oracle.attn_fwd_bwd(q, k, v, dO, cu, causal)
    ref = {"O": o, "dQ": dq, "dK": dk, "dV": dv}
    runs = [GpuAttn(ctx).run(q, k, v, dO, cu, causal=causal, grad_f32=grad_f32) for _ in range(2)]
    check_against_budget(f"{len(lens)} sequences", runs[0], ref, q, k, v, dO, cu, causal, None, grad_f32, stated)
    assert np.abs(runs[0]["LSE"] - lse).max() < 1e-3
    for name in runs[0]:
        assert np.array_equal(runs[0][name], runs[1][name]), name


# items per pass: half a chip, one and two workgroups per compute unit, and one more than each
@pytest.mark.parametrize("per_cu,more,heads,D", [(0.5, 0, 1, 128), (0.5, 1, 1, 128), (1, 0, 4, 128), (1, 1, 1, 128), (1, 1, 1, 64),
                                                 (2, -2, 1, 64), (2, 0, 1, 64), (2, 1, 1, 64), (2, 0, 4, 128), (2, 4, 4, 128)])
def test_items_around_the_lines(ctx, per_cu, more, heads, D):
    check(ctx, case_lengths(int(per_cu * ctx.num_cu) + more, heads), heads, heads, D, True)


@pytest.mark.parametrize("lens,hq,hkv,D,causal", [
    ([1], 1, 1, 128, True), ([300, 70], 1, 1, 128, False), ([300, 70], 3, 3, 64, True), ([513, 31], 8, 2, 128, True),
    ([511, 257], 8, 2, 64, False), ([1030], 4, 1, 128, True), ([1025, 64, 129], 2, 2, 128, False), ([1500], 2, 2, 64, True),
])
@pytest.mark.parametrize("grad_f32", [True, False])
def test_few_long_items(ctx, lens, hq, hkv, D, causal, grad_f32):
    check(ctx, lens, hq, hkv, D, causal, grad_f32)



@pytest.mark.parametrize("causal", [True, False])
def test_three_workgroups_per_unit(ctx, causal):
    """D = 64 and items that are short against a workgroup's share: forward, dQ and dK/dV (of 64 keys: walks are short) run three
    workgroups per compute unit."""
    # (the flat 2e-2 is a statement about the magnitudes of the configurations: among 7 million dV elements that sum four query
    # heads some are large enough for two or three roundings of P to bf16, 2^-8 of a term each, to pass it (2.1e-2 seen);
    # the budget that is derived element by element from those roundings holds)
    check(ctx, [200 + (37 * i) % 150 for i in range(150)], 16, 4, 64, causal, stated=False)
