"""Where every queue gets several heads of a sequence, they are neighbours: with grouped heads a queue's items read few key heads."""
import pytest

from paper_2412_01523_amd import binding as fx
from paper_2412_01523_amd import workloads as wl


@pytest.fixture(scope="module")
def host_ctx():
    c = fx.Context(-1)
    yield c
    c.close()


@pytest.mark.parametrize("hq,hkv", [(16, 2), (16, 1), (8, 2), (32, 4), (24, 3), (12, 4), (4, 1)])
@pytest.mark.parametrize("shard", [False, True])
def test_a_queue_holds_neighbouring_heads(host_ctx, hq, hkv, shard):
    lens = [4096]
    cu = wl.cu_seqlens(lens)
    plan = fx.ShardPlan(host_ctx, cu, cu, [0], hq, hkv, 128, False) if shard else fx.Plan(host_ctx, cu, hq, hkv, 128, False)
    for which in (fx.PASS_FWD, fx.PASS_BWD_DQ):
        items, offs = plan.items(which)
        assert sorted(set(zip(items["head"].tolist(), items["tile"].tolist()))) == [(h, t) for h in range(hq) for t in range(32)]
        if hq % 8:
            continue
        for x in range(8):
            heads = sorted(set(items["head"][int(offs[x]):int(offs[x + 1])].tolist()))
            assert heads == list(range(heads[0], heads[0] + hq // 8))
    plan.close()
