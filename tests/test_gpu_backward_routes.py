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
