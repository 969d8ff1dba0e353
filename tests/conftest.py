import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu where there is one)")


@pytest.fixture(scope="session")
def assembly(tmp_path_factory):
    """Device assembly of every translation unit with kernels: unit -> text."""
    from paper_2503_16672_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    units = sorted(f[:-4] for f in os.listdir(build.CSRC) if f.startswith("k_"))
    d = tmp_path_factory.mktemp("asm")

    def one(unit):
        out = d / f"{unit}.s"
        subprocess.run([build.HIPCC, *build.FLAGS, "-w", "--cuda-device-only", "-S", os.path.join(build.CSRC, f"{unit}.hip"), "-o", str(out)], check=True)
        return out.read_text()

    with ThreadPoolExecutor(len(units)) as ex:
        return dict(zip(units, ex.map(one, units)))
