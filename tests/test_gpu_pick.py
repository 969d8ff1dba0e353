"""The keep-2-of-4 pick of the activation epilogues on inputs where it can go wrong: few levels, so that most groups hold equal magnitudes
(ties go to the lower index), zeros of both signs, infinities and values next to each other at both ends of the bf16 range -- in every
block tile (test_tile_rule checks that the shapes take them), which pair the groups two by two in different ways.  X selects one row of W1
per token, so the pre-activation is a stored weight, exactly, and the pick is compared bit for bit with the oracle's on the rounded squares."""
import numpy as np
import pytest
import torch

import test_gpu_parity as P
from oracle import ffn24_oracle as O

pytestmark = pytest.mark.gpu
F24 = P.F24
ROWS = 256             # rows of W1 that tokens select; the others are zero
# T, D, F and the tile of the up-projection, of bf16 and of row-wise fp8 (0: 256 x 256, 1: 256 x 128, 2: 128 x 128, 3: 128 x 64, 4: 64 x 64)
SHAPES = [(256, 256, 768, 4), (256, 256, 1024, 4), (512, 256, 4096, 3), (1024, 256, 4096, 2), (2048, 256, 4096, 2), (4096, 256, 8192, 2), (1536, 768, 2816, 1), (2048, 1024, 4096, 1),
          (3328, 3584, 3840, 0)]
LEVELS = np.array([-2.0, -0.0, 0.0, 2.0 ** -60, 2.0 ** -80, 1.0, 1.0078125, 2.0, 2.015625, 3.0, 2.0 ** 63, 2.0 ** 70], np.float32)


def _weights(Fh, seed):
    """[ROWS, Fh] of LEVELS: uniform draws, with every fourth row made of two levels only and every eighth of one."""
    rng = np.random.default_rng(seed)
    W = LEVELS[rng.integers(0, len(LEVELS), size=(ROWS, Fh))]
    W[::4] = LEVELS[rng.integers(0, 2, size=W[::4].shape) * rng.integers(1, len(LEVELS), size=(len(W[::4]), 1))]
    W[::8] = LEVELS[rng.integers(0, len(LEVELS), size=(len(W[::8]), 1))]
    return W


def _expected(W):
    z = np.maximum(W, 0).astype(np.float32)
    with np.errstate(over="ignore"):
        h = z * z
    return O.sparsify24(O.f32_to_bf16_bits(h))


def _operands(W, T, D, seed):
    """X [T, D] of ones and zeros and W1 [D, Fh] with the rows of W spread over k, so that token t's row of X W1 is W[sel[t]]."""
    sel = np.random.default_rng(seed).integers(0, ROWS, size=T)
    X = torch.zeros((T, D))
    X[torch.arange(T), torch.from_numpy(sel * (D // ROWS))] = 1.0
    W1 = np.zeros((D, W.shape[1]), np.float32)
    W1[::D // ROWS] = W
    return X, W1, sel


@pytest.mark.parametrize("T,D,Fh,tile", SHAPES)
def test_pick_of_ties_and_extremes_bf16(F24, T, D, Fh, tile):
    print(f"pick bf16 T={T} D={D} F={Fh}", flush=True)
    W = _weights(Fh, T)
    X, W1, sel = _operands(W, T, D, 1)
    ctx = F24.Context(T, D, Fh)
    ctx.ffn24_fwd(X.to(torch.bfloat16).cuda(), P.to_dev_bf16(W1), None, torch.zeros((Fh, D), dtype=torch.bfloat16, device="cuda"))
    torch.cuda.synchronize()
    vals, meta = _expected(W)
    assert np.array_equal(ctx.saved("meta").cpu().numpy(), meta[sel])
    assert np.array_equal(ctx.saved("Hc").cpu().view(torch.int16).numpy().view(np.uint16), vals[sel])


@pytest.mark.parametrize("T,D,Fh,tile,counts", [(*q, c) for c in (False, True) for q in SHAPES if q[2] >= 1024 or not c])   # (a split needs 1024 features)
def test_pick_and_row_maxima_fp8_rowwise(F24, T, D, Fh, tile, counts):
    """The same with e4m3 operands and unit scales: levels an e4m3 weight holds; the row scale is the largest kept activation / 448.  With a split
    the epilogue also counts every feature's non-zero activations."""
    print(f"pick fp8 T={T} D={D} F={Fh} counts={counts}", flush=True)
    rng = np.random.default_rng(T + 1)
    W = np.array([-2.0, 0.0, 0.0, 1.0, 1.125, 2.0, 3.0, 0.5, 0.015625], np.float32)[rng.integers(0, 9, size=(ROWS, Fh))]
    W[::8] = 0.0
    X, W1, sel = _operands(W, T, D, T + 2)
    code = lambda t: t.to(torch.float8_e4m3fn).view(torch.uint8).cuda()
    one = lambda n: torch.ones(n, dtype=torch.float32, device="cuda")
    ctx = F24.Context(T, D, Fh, F24.FFN24_ROWWISE | F24.FFN24_TRAINING | (F24.FFN24_SPLIT if counts else 0), F24.FFN24_FP8_E4M3)
    ctx.set_row_scales(one(T), one(Fh), one(D))
    if counts:
        ctx.set_split(256)
    ctx.ffn24_fwd(code(X), code(torch.from_numpy(W1)), None, code(torch.zeros((Fh, D))))
    torch.cuda.synchronize()
    vals, meta = _expected(W)
    assert np.array_equal(ctx.saved("meta").cpu().numpy(), meta[sel])
    assert np.array_equal(ctx.saved("Hc16").cpu().view(torch.int16).numpy().view(np.uint16), vals[sel])
    mx = O.bf16_bits_to_f32(vals).max(axis=1)[sel].astype(np.float32)
    assert np.array_equal(ctx.saved("sh").cpu().numpy(), np.where(mx > 0, mx / np.float32(448), np.float32(1)))
    if counts:
        assert np.array_equal(ctx.saved("nnz").cpu().numpy(), (W > 0)[sel].sum(axis=0))
