"""dK/dV items of 128 keys (D = 64): edges of tiles, blocks and steps, walks of one, two, three and many steps, grouped heads, tiles
cut into parts, both gradient types, against the CPU fp64 oracle and the rounding budget."""
import numpy as np
import pytest

import oracle
from paper_2412_01523_amd import workloads as wl

from gpu_util import GpuAttn, check_against_budget

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 320, 384]


@pytest.mark.parametrize("lens,hq,hkv,causal,f32,cut", [
    (EDGES * 3, 4, 4, False, False, False), (EDGES + [2100, 449], 8, 4, False, True, True),
    ([65, 127, 128, 193, 255, 256, 321, 383, 384] * 4 + [449], 8, 4, False, True, False),
    ([1025, 1, 960, 1151, 0, 833, 1217] * 2, 4, 4, True, True, False), ([1537, 895, 1280, 700], 8, 8, True, False, False),
    ([4200, 2300, 65], 8, 1, True, False, True), ([2049, 1300, 700, 130], 8, 4, False, True, True),
], ids=["edges", "edges beside a long one, grouped", "edges, grouped", "causal", "causal, more heads", "causal, cut", "cut"])
def test_backward_with_128_key_items(lens, hq, hkv, causal, f32, cut):
    from paper_2412_01523_amd import binding as fx
    ctx = fx.Context(0)
    D, cu = 64, wl.cu_seqlens(lens)
    T = int(cu[-1])
    print(f"128-key items: {len(lens)} sequences, {hq} heads on {hkv}, causal={causal}, f32={f32}", flush=True)
    plan = fx.Plan(ctx, cu, hq, hkv, D, causal)
    assert plan.tile_rows(fx.PASS_BWD_DKV) == 128
    assert (plan.items(fx.PASS_BWD_DKV)[0]["nparts"] > 1).any() == cut
    plan.close()
    q, g = (wl.normal_bf16(931, tid, (T, hq, D)) for tid in (wl.TID_Q, wl.TID_DO))
    k, v = (wl.normal_bf16(931, tid, (T, hkv, D)) for tid in (wl.TID_K, wl.TID_V))
    O, _, dQ, dK, dV = oracle.attn_fwd_bwd(q, k, v, g, cu, causal)
    runs = [GpuAttn(ctx).run(q, k, v, g, cu, causal, grad_f32=f32) for _ in range(2)]
    for name in ("dQ", "dK", "dV"):
        assert np.array_equal(runs[0][name], runs[1][name]), f"{name} is not reproducible"
    check_against_budget("128 keys", runs[0], {"O": O, "dQ": dQ, "dK": dK, "dV": dV}, q, k, v, g, cu, causal, None, f32)
    ctx.close()
