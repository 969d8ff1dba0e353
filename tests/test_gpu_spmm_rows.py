"""spmm24 on row-major operands around the reduction length from which it takes slots of 128 k, with rows that end inside a slot and start
inside a line, in every tile.  Small integers, so that every sum is exact in fp32 and the result is equal to the rounded reference."""
import numpy as np
import pytest
import torch

import test_gpu_parity as P
from oracle import ffn24_oracle as O

pytestmark = pytest.mark.gpu
F24 = P.F24


@pytest.mark.parametrize("M,N", [(256, 256), (2048, 1024), (2048, 2048), (4096, 2048), (8192, 2048)])   # 64 x 64, 128 x 64, 128 x 128, 256 x 128, 256 x 256
@pytest.mark.parametrize("K", [1984, 2048, 2112, 2176, 2240])
def test_spmm24_slots_exact(F24, M, N, K):
    print(f"spmm24 slots M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A = rng.integers(-3, 4, size=(256, K)).astype(np.float32)
    B = rng.integers(-3, 4, size=(N, K)).astype(np.float32)
    vals, meta = O.sparsify24(O.f32_to_bf16_bits(A))
    ref = torch.from_numpy(np.asarray(P._mm24(O.bf16_bits_to_f32(vals).astype(np.float64), meta, B.T.astype(np.float64)), np.float32)).to(torch.bfloat16)
    rows = np.concatenate([np.roll(np.arange(256), i) for i in range(M // 256)])    # every block of 256 rows in another order
    C = F24.spmm24(P.dev_bf16_from_words(np.ascontiguousarray(vals[rows])), torch.from_numpy(np.ascontiguousarray(meta[rows])).cuda(), P.to_dev_bf16(B))
    torch.cuda.synchronize()
    assert torch.equal(C.cpu(), ref[torch.from_numpy(rows)])
