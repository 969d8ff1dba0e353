"""The 256 x 256 block tile, whose matrix ops are other instructions than the smaller tiles': reductions of fewer stages than its ring holds and just
beyond, exactly, and whole steps of every kind bit for bit against the same step in smaller tiles (a token's row of Y and dX depends on no
other token, a feature's part of dW1 and dW2 on no other feature group, and every tile sums the same k in the same order)."""
import numpy as np
import pytest
import torch

import test_gpu_parity as P
from oracle import ffn24_oracle as O
from test_gpu_tiles import _fp8_step

pytestmark = pytest.mark.gpu
F24 = P.F24


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 704])
def test_spmm24_short_reductions_exact(F24, K):
    """Small integers: every sum is exact in fp32, and bf16 rounds it once, so the result is equal to the rounded reference."""
    M = N = 4096
    print(f"spmm24 256 x 256 tiles K={K}", flush=True)
    rng = np.random.default_rng(K)
    A = rng.integers(-3, 4, size=(512, K)).astype(np.float32)
    B = rng.integers(-3, 4, size=(N, K)).astype(np.float32)
    vals, meta = O.sparsify24(O.f32_to_bf16_bits(A))
    ref = torch.from_numpy(np.asarray(P._mm24(O.bf16_bits_to_f32(vals).astype(np.float64), meta, B.T.astype(np.float64)), np.float32)).to(torch.bfloat16)
    rows = np.concatenate([np.roll(np.arange(512), 5 * i) for i in range(M // 512)])    # every block of rows in another order
    C = F24.spmm24(P.dev_bf16_from_words(np.ascontiguousarray(vals[rows])), torch.from_numpy(np.ascontiguousarray(meta[rows])).cuda(), P.to_dev_bf16(B))
    torch.cuda.synchronize()
    assert torch.equal(C.cpu(), ref[torch.from_numpy(rows)])


def _bf16_step(F24, dev, b1, dense, ts, fs):
    ctx = F24.Context(ts, dev["X"].shape[1], fs, F24.FFN24_TRAINING | (F24.FFN24_DENSE if dense else 0))
    X, W1, W2, dY = dev["X"][:ts].contiguous(), dev["W1"][:, :fs].contiguous(), dev["W2"][:fs].contiguous(), dev["dY"][:ts].contiguous()
    Y = (ctx.ffn_fwd if dense else ctx.ffn24_fwd)(X, W1, b1[:fs].contiguous(), W2)
    g = (ctx.ffn_bwd if dense else ctx.ffn24_bwd)(dY)
    torch.cuda.synchronize()
    ctx.close()
    return (Y, *g)


# (T, D, F): 256 x 256 tiles in every GEMM of every kind (test_tile_rule.py), less than a round of them; in all but the dense and the fp8 up- and
# down-projections and the dense fp8 weight gradients, an odd multiple of 256 as the short reduction and more than a round
SIZES = [(3584, 3584, 3584), (8192, 2304, 8192)]


@pytest.mark.parametrize("T,D,Fh", SIZES)
@pytest.mark.parametrize("kind", ["bf16", "fp8", "fp8_rowwise"])
@pytest.mark.parametrize("dense", [False, True])
def test_steps_have_the_bits_of_smaller_tiles(F24, kind, dense, T, D, Fh):
    g = torch.Generator(device="cuda").manual_seed(11)
    dev = {k: torch.randn(*s, generator=g, device="cuda") for k, s in (("X", (T, D)), ("W1", (D, Fh)), ("W2", (Fh, D)), ("dY", (T, D)))}
    b1 = torch.full((Fh,), -0.05, device="cuda")
    if kind == "bf16":
        dev["W1"] /= D ** 0.5
        dev["W2"] /= Fh ** 0.5
        dev = {k: v.bfloat16() for k, v in dev.items()}
        step = lambda ts, fs: _bf16_step(F24, dev, b1, dense, ts, fs)
    else:
        dev = {k: (v * 64).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) for k, v in dev.items()}
        q = {k: v for k, v in dev.items()}
        step = lambda ts, fs: _fp8_step(F24, q, dev, b1, kind == "fp8_rowwise", dense, ts, fs)
    print(f"256 x 256 tiles {kind} dense={dense} T={T} D={D} F={Fh}", flush=True)
    full = step(T, Fh)
    assert float(full[0].float().abs().max()) > 0 and all(bool(torch.isfinite(x.float()).all()) for x in full)
    got = step(512, Fh)
    assert torch.equal(got[0], full[0][:512]) and torch.equal(got[1], full[1][:512])
    if kind == "fp8_rowwise":
        return                                        # a token's scale is the maximum over all its features, so a slice of features has other scales
    got = step(T, 256)
    assert torch.equal(got[2], full[2][:, :256]) and torch.equal(got[3], full[3][:256])
