"""The forward in halves (few long sequences: two workgroups per item, each wavefront half of the keys): walks around the shortest that
is split, odd and even numbers of key tiles, ragged ends, a second half of a tile without rows, several sequences, grouped heads,
keys that make the wavefronts of one half recompute their rows.  Against the CPU fp64 oracle and the rounding budget, and with the
same bits with a plan and without."""
import numpy as np
import pytest

import oracle
from paper_2412_01523_amd import workloads as wl

from gpu_util import check_against_budget, to_bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,causal", [(128, True), (64, True), (128, False), (64, False)])
@pytest.mark.parametrize("lens,hq,hkv,outgrow", [
    ([512], 8, 8, None), ([513], 2, 1, None), ([575], 3, 3, None), ([833], 4, 2, None), ([1, 1700, 65], 2, 2, None),
    ([897, 640], 4, 1, None), ([1984], 3, 1, None), ([3000], 1, 1, None), ([1500], 2, 2, (1100, 48.0)), ([1500], 2, 2, (40, 64.0)),
], ids=lambda x: str(x).replace(" ", ""))
def test_forward_in_halves(lens, hq, hkv, outgrow, D, causal):
    _check(lens, hq, hkv, outgrow, D, causal)


def test_forward_in_halves_with_more_items_than_compute_units():
    """Short rows: a compute unit holds a workgroup and a half of the items' pairs before whole items are the better ones."""
    _check([1999], 16, 4, None, 64, True)


def _check(lens, hq, hkv, outgrow, D, causal):
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"forward in halves: {lens}, {hq} heads on {hkv}, D={D}, causal={causal}, {outgrow}", flush=True)
    ctx = fx.Context(0)
    cu, T = wl.cu_seqlens(lens), sum(lens)
    # the line the choice is made by (see fwd_halves): the cases lie on its near side
    items = (-(-T // 128) + len(lens)) * hq
    assert T >= 512 * len(lens) and (3 * items <= 2 * ctx.num_cu or D == 64 and ctx.num_cu < items and 2 * items <= 3 * ctx.num_cu)
    q = wl.normal_bf16(941, wl.TID_Q, (T, hq, D))
    k, v = (wl.normal_bf16(941, tid, (T, hkv, D)) for tid in (wl.TID_K, wl.TID_V))
    if outgrow:
        kf = wl.bf16_bits_to_f32(k)
        kf[outgrow[0]:] *= np.float32(outgrow[1])
        k = wl.f32_to_bf16_bits(kf)
    O, LSE, *_ = oracle.attn_fwd_bwd(q, k, v, q, cu, causal)
    qd, kd, vd, cud = to_dev(q), to_dev(k), to_dev(v), torch.from_numpy(cu).cuda()
    plan = fx.Plan(ctx, cu, hq, hkv, D, causal)
    whole = int(plan.items(fx.PASS_FWD)[0]["nparts"].max()) == 1
    runs = []
    for planned in (False, False, True):
        o = torch.full((T, hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, T), float("nan"), dtype=torch.float32, device="cuda")
        if planned:
            fx.flexsp_attn_varlen_fwd(ctx, plan, qd, kd, vd, cud, o, lse, causal=causal)
        else:
            fx.flexsp_attn_varlen_fwd_static(ctx, qd, kd, vd, cud, o, lse, causal=causal)
        runs.append((to_bits(o), lse.cpu().numpy()))
    plan.close()
    for o, lse in runs[1:2 + whole]:
        assert np.array_equal(o, runs[0][0]) and np.array_equal(lse, runs[0][1])
    # (fp32 spacing grows with |LSE|)
    assert np.abs(runs[0][1] - LSE).max() < 1e-3 * max(1.0, float(np.abs(LSE).max()) / 16)
    check_against_budget("halves", {"O": runs[0][0]}, {"O": O}, q, k, v, q, cu, causal, None, False, stated=not outgrow,
                         rel_l2=2e-2 if outgrow else 5e-3)
    ctx.close()
