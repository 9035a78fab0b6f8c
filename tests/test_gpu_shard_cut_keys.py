"""Backward of a key shard whose 64-key tiles are cut into parts: dealt, and one workgroup to an item, in one launch with the dQ pass
and apart from it; stored as bf16 and added to fp32 sums; against the oracle, and the same bits every time."""
import numpy as np
import pytest

import oracle
from paper_2412_01523_amd import workloads as wl

from gpu_util import MAX_ABS, REL_L2, bf16_f64, errors
from test_gpu_kvshard import _complete_statistics, _shard_backward, ctx  # noqa: F401

pytestmark = pytest.mark.gpu

#        query rows, shard keys, shift, heads, key heads, D, causal, tiles of the plan's own list are cut
CASES = {
    "dealt": ([1200] + [40] * 260, [1300] + [40] * 260, [0] + [0] * 260, 4, 2, 128, True, True),
    "dealt-d64-whole-shift": ([2100, 40] * 2, [1500, 64] * 2, [1500, 64] * 2, 8, 8, 64, True, False),
    "both-few-steps": ([513], [200], [100], 8, 1, 128, True, True),
    "both-d64-not-causal": ([640, 1], [129, 70], [0, 0], 6, 2, 64, False, False),
    "two-launches": ([4100], [700], [-300], 16, 2, 128, True, True),
    "rows-that-see-no-key": ([700], [900], [-500], 4, 1, 128, True, False),
}


@pytest.mark.parametrize("name", CASES)
def test_cut_key_tiles(ctx, name):  # noqa: F811
    from paper_2412_01523_amd import binding as fx
    lq, lk, shift, Hq, Hkv, D, causal, listed = CASES[name]
    print(f"shard backward, cut key tiles: {name}", flush=True)
    cu_q, cu_k = wl.cu_seqlens(lq), wl.cu_seqlens(lk)
    plan = fx.ShardPlan(ctx, cu_q, cu_k, shift, Hq, Hkv, D, causal)
    assert (plan.items(fx.PASS_BWD_DKV)[0]["nparts"] > 1).any() == listed
    plan.close()
    q = wl.normal_bf16(6200, wl.TID_Q, (sum(lq), Hq, D)); g = wl.normal_bf16(6200, wl.TID_DO, (sum(lq), Hq, D))
    k = wl.normal_bf16(6200, wl.TID_K, (sum(lk), Hkv, D)); v = wl.normal_bf16(6200, wl.TID_V, (sum(lk), Hkv, D))
    O, LSE = _complete_statistics(q, k, v, cu_q, cu_k, shift, causal, 13, 6200)
    ref = oracle.attn_bwd_kvshard(q, k, v, g, LSE, np.einsum("thd,thd->ht", bf16_f64(g), O), cu_q, cu_k, shift, causal)
    o_bits = wl.f32_to_bf16_bits(O.astype(np.float32))
    rng = np.random.default_rng(62)
    before = [rng.standard_normal(x.shape).astype(np.float32) for x in ref]
    for onto in (None, before):
        runs = [_shard_backward(ctx, q, k, v, o_bits, g, LSE, cu_q, cu_k, shift, causal, onto is not None, onto) for _ in range(2)]
        for i, (n, want) in enumerate(zip(("dQ", "dK", "dV"), ref)):
            assert np.array_equal(runs[0][i], runs[1][i]), f"{n} is not reproducible"
            got = runs[0][i] - (before[i] if onto else 0.0)
            top = float(np.abs(want).max(initial=0.0))  # (a shard of few keys that many rows see: the bound is a share of its largest value)
            ma, rl = errors(got, want)
            print(f"  {n} {'added' if onto else 'stored'}: max_abs={ma:.2e} rel_l2={rl:.2e} (largest value {top:.1f})", flush=True)
            assert (np.abs(got - want) <= max(MAX_ABS, REL_L2 * top) + (0.0 if onto else np.abs(want) * 2.0 ** -8)).all(), n
            assert rl <= REL_L2 or n == "dQ", n  # (dQ is a part of the rows' gradient, its error that of the whole)
