"""Launches of few items, where the kernels are started one workgroup per item, and the sizes around the line where
they become persistent (two workgroups per compute unit): against the CPU fp64 oracle, twice through one plan."""
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


@pytest.mark.parametrize("around,heads,D", [(-2, 1, 64), (0, 1, 64), (1, 1, 64), (0, 4, 128), (4, 4, 128), (None, 1, 128), (None, 3, 64)])
@pytest.mark.parametrize("causal", [True, False])
def test_items_around_the_persistent_line(ctx, around, heads, D, causal):
    lens = [300, 70] if around is None else case_lengths(2 * ctx.num_cu + around, heads)
    print(f"launch shape: {len(lens)} sequences x {heads} heads, D={D}, causal={causal}", flush=True)
    cu = wl.cu_seqlens(lens)
    T = int(cu[-1])
    q, k, v, dO = (wl.normal_bf16(911, tid, (T, heads, D)) for tid in (wl.TID_Q, wl.TID_K, wl.TID_V, wl.TID_DO))
    o, lse, dq, dk, dv = oracle.attn_fwd_bwd(q, k, v, dO, cu, causal)
    ref = {"O": o, "dQ": dq, "dK": dk, "dV": dv}
    runs = [GpuAttn(ctx).run(q, k, v, dO, cu, causal=causal, grad_f32=True) for _ in range(2)]
    check_against_budget(f"{len(lens)} sequences", runs[0], ref, q, k, v, dO, cu, causal, None, True)
    assert np.abs(runs[0]["LSE"] - lse).max() < 1e-3
    for name in runs[0]:
        assert np.array_equal(runs[0][name], runs[1][name]), name
