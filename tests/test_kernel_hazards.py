"""The matrix ops of the 256 x 256 tiles are inline assembly, for which the compiler adds no wait states (no GPU): no vector instruction may write an
operand of a matrix op within the two instructions before it, in any GEMM kernel."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

import pytest

from paper_2503_16672_amd import build

SRC = Path(build.CSRC)
UNITS = ["k_fwd", "k_bwd", "k_wgrad", "k_dense_a", "k_dense_b", "k_fp8", "k_fp8_rowwise"]
WAIT = 2


def _registers(operand):
    m = re.fullmatch(r"([va])(\d+)|([va])\[(\d+):(\d+)\]", operand)
    if not m:
        return set()
    return {(m[1], int(m[2]))} if m[1] else {(m[3], i) for i in range(int(m[4]), int(m[5]) + 1)}


def _hazards(text):
    """(matrix ops, those with an operand written too shortly before)"""
    ops, bad, before = 0, [], []                       # before: (wait states an instruction is worth, vector registers it writes)
    for line in text.splitlines():
        x = line.split(";")[0].strip()
        if not x or x[0] == "." or x.endswith(":"):
            continue
        name, _, rest = x.partition(" ")
        operands = [a.strip().split(" ")[0] for a in rest.split(",")]
        matrix = "mfma" in name or "smfmac" in name
        if matrix:
            ops += 1
            used, waited = set().union(*map(_registers, operands)), 0
            for states, written in reversed(before):
                if waited >= WAIT:
                    break
                if written & used:
                    bad.append(x)
                waited += states
        states = int(rest.split()[0]) + 1 if name == "s_nop" else 1
        before = before[-3:] + [(states, _registers(operands[0]) if name.startswith("v_") and not matrix else set())]
    return ops, bad


@pytest.mark.parametrize("unit", UNITS)
def test_no_operand_is_written_right_before_a_matrix_op(assembly, unit):
    ops, bad = _hazards(assembly[unit])
    assert ops > 500 and not bad, (unit, ops, bad[:5])


def test_the_check_finds_a_hazard():
    near = "v_mov_b32_e32 v5, v9\n\ts_nop 0\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[2:5], v[6:9], a[0:3]\n"
    far = near.replace("s_nop 0", "s_nop 1")
    assert len(_hazards(near)[1]) == 1 and _hazards(far) == (1, [])


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("asm")

    def one(unit):
        out = d / f"{unit}.s"
        subprocess.run([build.HIPCC, *build.FLAGS, "-w", "--cuda-device-only", "-S", str(SRC / f"{unit}.hip"), "-o", str(out)], check=True)
        return out.read_text()

    with ThreadPoolExecutor(len(UNITS)) as ex:
        return dict(zip(UNITS, ex.map(one, UNITS)))
