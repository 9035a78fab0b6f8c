"""CPU: what the compiler says about the forward kernels' registers."""
import re
import subprocess

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


def test_forward_kernels_hardly_spill():
    """A spilled vector register is a trip to scratch memory, and the shard forward's lie in the stretch that every item runs
    through.  29 is what its D = 128 variant spills (some tens more have cost short items half their time), 16 the plain one's."""
    src = "attn_fwd.hip"
    r = subprocess.run([build._hipcc(), *build.FLAGS, *build.PER_SOURCE[src], "-Rpass-analysis=kernel-resource-usage",
                        "--cuda-device-only", "-c", str(build.CSRC / src), "-o", "/dev/null"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spills = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert len(names) == len(spills) >= 6, r.stderr[-3000:]
    print(dict(zip(names, spills)))
    assert max(spills) <= 32, dict(zip(names, spills))
