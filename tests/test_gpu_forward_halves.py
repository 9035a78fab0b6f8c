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


@pytest.mark.parametrize("lens,hq,hkv,D", [([5000], 4, 2, 64), ([2100, 2300], 4, 4, 128)])
def test_forward_in_halves_with_more_workgroups_than_compute_units(lens, hq, hkv, D):
    """Under a mask, long sequences."""
    _check(lens, hq, hkv, None, D, True)


@pytest.mark.parametrize("lens,hq,hkv,D,causal", [([2176], 8, 2, 128, False), ([1408], 12, 3, 128, True), ([590, 433], 4, 4, 64, True),
                                                  ([2300], 8, 4, 64, False)])
def test_whole_items_beyond_the_lines(lens, hq, hkv, D, causal):
    _check(lens, hq, hkv, None, D, causal, halves=False)


def _check(lens, hq, hkv, outgrow, D, causal, halves=True):
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"forward in halves: {lens}, {hq} heads on {hkv}, D={D}, causal={causal}, {outgrow}", flush=True)
    ctx = fx.Context(0)
    cu, T = wl.cu_seqlens(lens), sum(lens)
    plan = fx.Plan(ctx, cu, hq, hkv, D, causal)
    whole = int(plan.items(fx.PASS_FWD)[0]["nparts"].max()) == 1
    q = wl.normal_bf16(941, wl.TID_Q, (T, hq, D))
    k, v = (wl.normal_bf16(941, tid, (T, hkv, D)) for tid in (wl.TID_K, wl.TID_V))
    if outgrow:
        kf = wl.bf16_bits_to_f32(k)
        kf[outgrow[0]:] *= np.float32(outgrow[1])
        k = wl.f32_to_bf16_bits(kf)
    O, LSE, *_ = oracle.attn_fwd_bwd(q, k, v, q, cu, causal)
    qd, kd, vd, cud = to_dev(q), to_dev(k), to_dev(v), torch.from_numpy(cu).cuda()
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
    for o, lse in runs[0::2]:
        # (fp32 spacing grows with |LSE|)
        assert np.abs(lse - LSE).max() < 1e-3 * max(1.0, float(np.abs(LSE).max()) / 16)
        check_against_budget("halves", {"O": o}, {"O": O}, q, k, v, q, cu, causal, None, False, stated=not outgrow,
                             rel_l2=2e-2 if outgrow else 5e-3)
    # which way it ran: all keys as one shard are a forward in whole items, and halves round their probabilities against other
    # references (where a row has one key that counts there is nothing to round)
    shard = fx.ShardPlan(ctx, cu, cu, [0] * len(lens), hq, hkv, D, causal)
    if not outgrow and int(shard.items(fx.PASS_FWD)[0]["nparts"].max()) == 1:
        o = torch.empty((T, hq, D), dtype=torch.bfloat16, device="cuda")
        lse = torch.empty((hq, T), dtype=torch.float32, device="cuda")
        fx.flexsp_attn_varlen_fwd_kvshard(ctx, shard, qd, kd, vd, o, lse, causal=causal)
        same = np.array_equal(to_bits(o), runs[0][0])
    else:
        same = not halves
    shard.close()
    ctx.close()
    assert same == (not halves)
