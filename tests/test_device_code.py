"""What the compiler cannot check in the device code: csrc/factor.h updates a column with a multiply-add that reads its first operand
across lanes (DPP), written as inline assembly.  Such a read needs two instructions, or wait states, between it and whatever wrote the
operand; the compiler adds them to its own cross-lane reads but does not see this one.  The code gives it what it needs by its
order, and this test looks at what was made of that, copies that the compiler may have put in front included."""
import os
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2507_08143_amd import build as B

WAIT_STATES = 2


def _registers(operand):
    m = re.match(r"-?\|?([va])(\d+)$|-?\|?([va])\[(\d+):(\d+)\]$", operand)
    if not m:
        return set()
    kind = m.group(1) or m.group(3)
    first, last = (m.group(2), m.group(2)) if m.group(1) else (m.group(4), m.group(5))
    return {(kind, r) for r in range(int(first), int(last) + 1)}


def too_early(assembly):
    """-> (cross-lane multiply-adds seen, those that read what one of the two instructions before has written, or that stand so
    close behind a label that it cannot be told)"""
    seen, early, before = 0, [], []          # before: (registers written, wait states), the last first; None at a label
    for number, line in enumerate(assembly.split("\n"), 1):
        line = line.split(";")[0].split("//")[0].strip()
        if not line or (line.startswith(".") and not line.endswith(":")):
            continue
        if line.endswith(":"):
            before.insert(0, None)
            continue
        name, _, rest = line.partition(" ")
        operands = [o.strip() for o in rest.split(",")]
        if name.startswith("v_fmac_f64") and "row_newbcast" in line:
            seen += 1
            wanted, states = _registers(operands[1].split()[0]), 0
            assert wanted, line
            for entry in before:
                if states >= WAIT_STATES:
                    break
                if entry is None or entry[0] & wanted:
                    early.append((number, line))
                    break
                states += entry[1]
        writes = set()
        if name.startswith("v_"):
            writes = _registers(operands[0].split()[0])
            if name.startswith("v_swap"):
                writes |= _registers(operands[1].split()[0])
        before.insert(0, (writes, int(operands[0], 0) + 1 if name == "s_nop" else 1))
        del before[8:]
    return seen, early


def test_the_scan_sees_what_stands_too_close():
    read = "v_fmac_f64_dpp v[8:9], -v[2:3], v[4:5] row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
    write, other = "v_mul_f64 v[2:3], v[6:7], v[0:1]\n", "v_add_f64 v[6:7], v[6:7], v[0:1]\n"
    assert too_early(write + other + other + read) == (1, [])
    assert too_early(write + "s_nop 1\n" + read) == (1, [])
    assert too_early(other + other + read + read) == (2, [])
    for bad in (write + read, write + other + read, write + "s_nop 0\n" + read, "v_mov_b32_e32 v3, v1\n" + other + read,
                "v_accvgpr_read_b32 v2, a7 ; reload\n" + other + read, ".LBB0_1:\n" + other + read):
        assert len(too_early(bad)[1]) == 1, bad


@pytest.fixture(scope="module")
def assemblies(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm")

    def compile_one(src):
        path = str(out / (src + ".s"))
        B._run([B.HIPCC, *B.FLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", path])
        return open(path).read()

    with ThreadPoolExecutor(max_workers=2) as ex:
        return dict(zip(("score.hip", "solve.hip"), ex.map(compile_one, ("score.hip", "solve.hip"))))


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="no hipcc")
@pytest.mark.parametrize("src", ["score.hip", "solve.hip"])
def test_cross_lane_operands_are_not_written_just_before(assemblies, src):
    seen, early = too_early(assemblies[src])
    assert seen > 500
    assert not early, early[:5]
