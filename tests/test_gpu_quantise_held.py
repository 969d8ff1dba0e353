"""quantise_e4m3 per column where one workgroup holds a whole strip of columns: row counts on both sides of its sizes, column counts that leave a
strip (32 columns) or a round over the 8 XCDs unfinished; against the oracle, bit for bit.  And wide matrices on both sides of the rule that
takes it, also with a single slab of rows (64): the same codes and scales as column by column in pieces of 8192, which are always held."""
import numpy as np
import pytest
import torch

from oracle import ffn24_oracle as O
from paper_2503_16672_amd import ffn24

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [1, 255, 257, 512, 513, 1536, 1537])
@pytest.mark.parametrize("C", [8, 32, 264, 1032])
def test_columns(R, C):
    rng = np.random.default_rng(R * 7 + C)
    x = O.round_bf16((rng.standard_normal((R, C)) * np.exp(rng.uniform(-4, 4, size=(1, C)))).astype(np.float32))
    x[:, C // 2] = 0
    x[R - 1, 0] = 300.0                                # the last row holds a column's largest
    codes, scales = ffn24.quantise_e4m3(torch.from_numpy(x).cuda().to(torch.bfloat16), 0)
    want, s = O.quantise_rows_e4m3(np.ascontiguousarray(x.T))
    assert np.array_equal(scales.cpu().numpy(), s) and np.array_equal(codes.cpu().numpy(), want.T)


@pytest.mark.parametrize("R,C", [(1, 16384), (1, 16392), (8, 1 << 20), (64, 16424), (65, 16424), (512, 16384), (512, 16416), (640, 16384), (641, 8200), (1024, 8200), (1024, 24576), (1536, 8200),
                                 (1536, 16384), (1536, 45000)])
def test_wide_columns(R, C):
    g = torch.Generator(device="cuda").manual_seed(R + C)
    x = torch.empty(R, C, device="cuda").normal_(generator=g).mul_(torch.exp2(torch.arange(C, device="cuda") % 17 - 8.0)).to(torch.bfloat16)
    x[:, 5] = 0
    x[R - 1, C - 1] = 300.0
    codes, scales = ffn24.quantise_e4m3(x, 0)
    assert float(scales[C - 1]) == np.float32(300.0) / np.float32(448.0) and float(scales[5]) == 1.0
    for lo in range(0, C, 8192):
        want, s = ffn24.quantise_e4m3(x[:, lo:lo + 8192].contiguous(), 0)
        assert torch.equal(scales[lo:lo + 8192], s) and torch.equal(codes[:, lo:lo + 8192], want)
