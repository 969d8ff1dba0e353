"""quantise_e4m3 at the largest row count its entry point takes, 2^24, with rows that a whole workgroup shares: one workgroup a row is 2^32
work items in one grid dimension, one more than a launch may have.  The matrix (138 GB) repeats a block of rows, so that its codes
repeat the block's."""
import pytest
import torch

import test_gpu_parity as P

pytestmark = pytest.mark.gpu
F24 = P.F24


def test_most_rows_of_more_than_4096_columns(F24):
    R, C, B = 1 << 24, 4104, 4096
    torch.cuda.empty_cache()
    need = 3 * R * C + 4 * R + (8 << 30)
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip(f"needs {need >> 30} GiB of device memory")
    print(f"quantise_e4m3 R={R} C={C}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(24)
    block = torch.empty(B, C, device="cuda").normal_(generator=g).mul_(torch.exp2(torch.arange(B, device="cuda") % 13 - 6.0)[:, None]).bfloat16()
    block[7] = 0
    codes0, scales0 = F24.quantise_e4m3(block, 1)
    X = torch.empty(R // B, B, C, dtype=torch.bfloat16, device="cuda")
    X.copy_(block)
    codes, scales = F24.quantise_e4m3(X.view(R, C), 1)
    torch.cuda.synchronize()
    assert torch.equal(scales.view(R // B, B), scales0.expand(R // B, B))
    for i in range(0, R // B, 64):      # 64 blocks at a time: the comparison's own memory
        assert bool((codes.view(R // B, B, C)[i:i + 64] == codes0).all())
    del X, codes
    torch.cuda.empty_cache()
