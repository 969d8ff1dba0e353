"""The feature partition of a row-wise fp8 split runs in the launch that quantises dZ, up to a number of features, and by itself with profiling on: the
same bits on both sides of that line, with one and with several workgroups of the quantisation."""
import pytest
import torch

import test_gpu_parity as P
from test_gpu_profiling import _step

pytestmark = pytest.mark.gpu
F24 = P.F24


@pytest.mark.parametrize("T,Fh", [(256, 1024), (768, 1280), (256, 16384), (256, 16640)])
def test_partition_beside_the_quantisation(F24, T, Fh):
    ctx, step, _keep = _step(F24, "fp8 rowwise split", T, 256, Fh)
    together = step()
    rows = ctx.saved("feat_of_row").clone()
    ctx.set_profiling(True)
    apart = step()
    torch.cuda.synchronize()
    assert torch.equal(rows, ctx.saved("feat_of_row")) and rows.unique().numel() == Fh
    assert all(torch.equal(a, b) for a, b in zip(together, apart, strict=True))
    ctx.close()
