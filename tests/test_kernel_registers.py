"""Register use of the GEMM kernels, from the compiler's own report (no GPU): these keep everything in registers.  One spilled register gives a
kernel a scratch segment, which cost every tile of the sparse store kernels 0.15-0.2 us."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

import pytest

from paper_2503_16672_amd import build

SRC = Path(build.CSRC)
UNITS = ["k_fwd", "k_bwd", "k_fp8_rowwise"]


# translation unit, 2:4 operand, epilogue as the mangled name has it, wave tiles (4 x 4: 256 x 256, 4 x 2: 256 x 128)
@pytest.mark.parametrize("unit,sparse,epilogue,tiles", [
    ("k_fwd", 1, "11EpiRowMajorE", [(4, 4)]),
    ("k_fwd", 1, "17EpiRowMajorMappedE", [(4, 4)]),
    ("k_fwd", 0, "11EpiPrune24TILb0EE", [(4, 4), (4, 2)]),
    ("k_fwd", 0, "11EpiPrune24TILb1EE", [(4, 4), (4, 2)]),              # with the per-feature counts
    ("k_bwd", 0, "10EpiDGatherE", [(4, 4), (4, 2)]),
    ("k_fp8_rowwise", 0, "13EpiPrune24RwTILb0EE", [(4, 4), (4, 2)]),    # with row maxima
    ("k_fp8_rowwise", 0, "13EpiPrune24RwTILb1EE", [(4, 4), (4, 2)]),    # ... and the per-feature counts
    ("k_fp8_rowwise", 0, "12EpiDGatherRwE", [(4, 4), (4, 2)]),
])
def test_kernels_do_not_spill(report, unit, sparse, epilogue, tiles):
    for mi, ni in tiles:
        found = [k for k in report[unit] if f"gemm_kernelILb{sparse}E" in k and epilogue in k and f"Li0ELi{mi}ELi{ni}E" in k]
        assert len(found) == 1, found
        assert report[unit][found[0]] == (0, 0), (found[0], report[unit][found[0]])


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    """translation unit -> kernel name -> (spilled registers, bytes of scratch a work item)"""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("asm")

    def one(unit):
        out = d / f"{unit}.s"
        subprocess.run([build.HIPCC, *build.FLAGS, "-w", "--cuda-device-only", "-S", str(SRC / f"{unit}.hip"), "-o", str(out)], check=True)
        kernels = {}
        for m in re.finditer(r"\.name:\s+(_Z\S+)\n(.*?)\.vgpr_spill_count:\s+(\d+)", out.read_text(), re.S):
            kernels[m[1]] = (int(m[3]), int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", m[2])[1]))
        return kernels

    with ThreadPoolExecutor(len(UNITS)) as ex:
        return dict(zip(UNITS, ex.map(one, UNITS)))
