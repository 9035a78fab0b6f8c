"""CPU: the list of a backward in one pass and when there is one, who draws which item of it, and the memory plans take, keep and give back
(tests/sanitize/driver_chain.cpp, driver_dealer.cpp and driver_pool.cpp include the host source), under the sanitizers; what the compiler says about its kernels' registers."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2412_01523_amd import build
from test_sanitizers import OUT, ROOT, SAN, _run


def _run_driver(name):
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not found")
    OUT.mkdir(exist_ok=True)
    exe = OUT / name
    _run([hipcc, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17", "-fno-omit-frame-pointer",
          "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-fno-gpu-rdc",
          f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2412_01523_amd' / 'csrc'}", "-o", str(exe),
          str(SAN / f"{name}.cpp"), "-fsanitize=address", "-fsanitize=undefined"])
    assert "ok" in _run([str(exe)])


def test_lists_under_asan_ubsan():
    _run_driver("driver_chain")


def test_plan_memory_under_asan_ubsan():
    _run_driver("driver_pool")


def test_every_item_once_and_every_wait_ends():
    _run_driver("driver_dealer")


def test_registers():
    """Two wavefronts to a SIMD, nothing spilled to memory."""
    src = "attn_bwd_chain.hip"
    r = subprocess.run([build._hipcc(), *build.FLAGS, *build.PER_SOURCE[src], "-Rpass-analysis=kernel-resource-usage",
                        "--cuda-device-only", "-c", str(build.CSRC / src), "-o", "/dev/null"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    use = [[int(n) for n in re.findall(rf" {what}: (\d+)", r.stderr)]
           for what in ("VGPRs Spill", r"ScratchSize \[bytes/lane\]", "AGPRs", r"Occupancy \[waves/SIMD\]")]
    assert use[:3] == [[0, 0]] * 3 and len(use[3]) == 2 and min(use[3]) >= 2, use
