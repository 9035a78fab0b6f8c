"""CPU: what the compiler says about the attention kernels' registers."""
import re
import subprocess

import pytest

from paper_2412_01523_amd import build


def test_halves_hold_no_merge_of_cut_tiles():
    """The merge counts arrivals with an atomic and has barriers that half of a forward in halves would not reach: it must not be there,
    not only be out of reach of the lists."""
    src = "attn_fwd.hip"
    r = subprocess.run([build._hipcc(), *build.FLAGS, *build.PER_SOURCE[src], "--cuda-device-only", "-S", "-c", str(build.CSRC / src), "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    bodies = dict(re.findall(r"^(\S*attn_fwd_kernel\S*): *;[^\n]*\n(.*?)^\s*s_endpgm", r.stdout, re.M | re.S))
    halves = [n for n in bodies if "Li2EEE" in n]
    assert len(halves) == 2 and len(bodies) > 4, list(bodies)
    for n, body in bodies.items():
        assert ("atomic" in body) == (n not in halves and "ELb1ELi1" not in n), n  # (without a list whole items have none either)


@pytest.mark.parametrize("src,kernels,three_fit", [
    ("attn_fwd.hip", 13, r"attn_fwd_kernelILi64ELb0ELb[01]ELi1E"), ("attn_fwd_search.hip", 3, r"attn_fwd_search_kernelILi64E"),
    ("attn_bwd.hip", 13, r"attn_bwd_(dq|dkv)_kernelILi64E")])
def test_attention_kernels_keep_their_registers(src, kernels, three_fit):
    """A spilled vector register is a trip to scratch memory: none (some kernels use 250 or more of 256, the shard forward all of them).  Where
    the host launches three workgroups per compute unit (D = 64: forward, dQ and dK/dV of 64 keys) three have to fit, and do where the forward finds its items;
    elsewhere two, but for forwards in halves that have a unit to themselves.  No kernel keeps results of matrix instructions in the other half of the register file,
    which the vector unit does not reach."""
    r = subprocess.run([build._hipcc(), *build.FLAGS, *build.PER_SOURCE[src], "-Rpass-analysis=kernel-resource-usage",
                        "--cuda-device-only", "-c", str(build.CSRC / src), "-o", "/dev/null"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    use = list(zip(re.findall(r"Function Name: (\S+)", r.stderr), *(
        [int(n) for n in re.findall(rf" {what}: (\d+)", r.stderr)]
        for what in ("VGPRs Spill", r"Occupancy \[waves/SIMD\]", "AGPRs", r"ScratchSize \[bytes/lane\]"))))
    print(*use, sep="\n")
    assert len(use) == kernels
    three = [u for u in use if re.search(three_fit, u[0])]
    assert len(three) == {"attn_fwd.hip": 2, "attn_fwd_search.hip": 1, "attn_bwd.hip": 4}[src] and all(occupancy >= 3 for _, _, occupancy, _, _ in three), three
    for name, spilled, occupancy, agprs, scratch in use:
        assert spilled == 0 and scratch == 0 and agprs == 0, name
        assert occupancy >= (1 if re.search(r"attn_fwd_kernelILi128ELb0ELb0ELi2E|attn_fwd_either_kernelILi128ELi2E", name) else 2), name
