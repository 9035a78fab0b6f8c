"""CPU: the FLOPs bench.py credits to the kernels of a step are the step's, whichever way the backward was launched."""
import pytest

import bench
from paper_2412_01523_amd import workloads as wl


@pytest.mark.parametrize("launched", [("fwd", "bwd_dkv", "bwd_dq"), ("fwd", "bwd_dkv")], ids=["two launches", "one launch"])
def test_kernel_flops_add_up(launched):
    lens, heads, d = [17, 64, 100, 255], 4, 64
    flops = bench.kernel_flops(d, wl.causal_pairs(lens) * heads, launched)
    fwd, bwd = wl.attn_flops(lens, heads, d, True)
    assert set(flops) == set(launched)
    assert flops["fwd"] == fwd and sum(flops.values()) - flops["fwd"] == bwd
