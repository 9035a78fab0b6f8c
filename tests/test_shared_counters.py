"""CPU: the counters that forwards without a plan share are clear again after launches that overlapped (tests/sanitize/driver_leave.cpp
runs the count of leaving workgroups with others acting between its accesses), under the sanitizers."""
import os
import shutil

import pytest

from test_sanitizers import OUT, ROOT, SAN, _run


def test_overlapping_launches_leave_the_counters_clear():
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not found")
    OUT.mkdir(exist_ok=True)
    exe = OUT / "driver_leave"
    _run([hipcc, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17", "-fno-omit-frame-pointer",
          "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-fno-gpu-rdc",
          f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2412_01523_amd' / 'csrc'}", "-o", str(exe),
          str(SAN / "driver_leave.cpp"), "-fsanitize=address", "-fsanitize=undefined"])
    assert "ok" in _run([str(exe)])
