"""quantise_e4m3 per column where one workgroup holds a whole strip of columns: row counts on both sides of its sizes, column counts that leave a
strip (32 columns) or a round over the 8 XCDs unfinished; against the oracle, bit for bit."""
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
