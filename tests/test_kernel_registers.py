"""Register use of the GEMM kernels, from the compiler's own report (no GPU): the sparse 256 x 256 kernels with a plain store or a scattered
one keep everything in registers.  One spilled register gives a kernel a scratch segment, which cost every tile 0.15-0.2 us."""
import os
import re
import subprocess
from pathlib import Path

import pytest

from paper_2503_16672_amd import build

SRC = Path(build.CSRC)


@pytest.mark.parametrize("epilogue", ["EpiRowMajorE", "EpiRowMajorMappedE"])
def test_sparse_store_kernels_do_not_spill(report, epilogue):
    found = [k for k in report if "gemm_kernelILb1E" in k and epilogue in k and "Li4ELi4E" in k]
    assert len(found) == 1
    assert report[found[0]] == (0, 0)


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    """kernel name -> (spilled registers, bytes of scratch a work item) of the forward translation unit"""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("asm") / "k_fwd.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-w", "--cuda-device-only", "-S", str(SRC / "k_fwd.hip"), "-o", str(out)], check=True)
    kernels = {}
    for m in re.finditer(r"\.name:\s+(_Z\S+)\n(.*?)\.vgpr_spill_count:\s+(\d+)", out.read_text(), re.S):
        kernels[m[1]] = (int(m[3]), int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", m[2])[1]))
    return kernels
