"""CPU: wait states that neither the hardware nor, around inline assembly, the compiler keeps: five between a vector instruction that writes a scalar
register (v_readfirstlane, v_readlane of a spilled scalar) and a memory instruction that takes its address from it."""
import re
import subprocess

import pytest

from paper_2412_01523_amd import build

NEEDED = 5


def listing(src):
    """[(operation, operands)] of the source as compiled into the library, in the order of the code."""
    r = subprocess.run([build._hipcc(), *build.FLAGS, *build.PER_SOURCE.get(src, []), "--cuda-device-only", "-S", str(build.CSRC / src), "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    out = []
    for line in r.stdout.splitlines():
        line = line.split(";")[0].strip()
        if line and line[0] != "." and not line.endswith(":"):
            op, _, rest = line.partition(" ")
            out.append((op, re.split(r"[,\s]+", rest.strip())))
    return out


def scalars(operands):
    regs = set()
    for o in operands:
        m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", o)
        if m:
            regs |= {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))
    return regs


def too_early(code):
    """The memory instructions of a listing that take a scalar address too early (what lies in front in the listing; a jump is no shorter)."""
    found = []
    for at, (op, operands) in enumerate(code):
        if not re.match(r"global_|buffer_|flat_|scratch_", op):
            continue
        regs, waits = scalars(operands), 0
        for before, to in reversed(code[max(0, at - NEEDED):at]):
            if waits >= NEEDED or before == "s_endpgm":
                break
            if before.startswith("v_") and regs & scalars(to[:2 if "_co_" in before else 1]):
                found.append((before, to, op, operands, waits))
            waits += int(to[0]) + 1 if before == "s_nop" else 1
    return found


def test_it_finds_one():
    early = [("v_readlane_b32", ["s7", "v255", "17"]), ("s_mov_b32", ["m0", "s3"]), ("s_nop", ["0"]), ("global_load_lds_dwordx4", ["v1", "s[6:7]"])]
    assert len(too_early(early)) == 1
    assert not too_early([early[0], early[1], ("s_nop", ["3"]), early[3]])
    assert not too_early([early[0], ("s_nop", ["1"]), ("v_mov_b32_e32", ["v3", "v4"]), early[1], early[2], early[3]])


@pytest.mark.parametrize("src", [s for s in build.SOURCES if s != "flexsp_host.hip"])
def test_scalar_addresses(src):
    code = listing(src)
    assert not too_early(code)
    if src == "attn_bwd_chain.hip":  # the kernel whose scalars wait in lanes: whatever stands in front of them, its copies count for themselves
        copies = [at for at, (op, operands) in enumerate(code) if op.startswith("global_load_lds") and scalars(operands)]
        assert len(copies) >= 20
        for at in copies:
            waits, before = 0, at
            while waits < NEEDED and (code[before - 1][0] in ("s_nop", "global_load_lds_dwordx4") or "m0" in code[before - 1][1][:1]):
                before -= 1
                waits += int(code[before][1][0]) + 1 if code[before][0] == "s_nop" else 1
            assert waits >= NEEDED, code[before - 1:at + 1]
