"""With profiling on a backward takes its weight gradients from a launch each, without it from one for both where that is better: the same
bits either way, for every kind of backward, at shapes whose gradients take the smallest tiles, mixed ones, and 256 x 256 tiles together and
apart."""
import pytest
import torch

import test_gpu_parity as P

pytestmark = pytest.mark.gpu
F24 = P.F24

# weight gradients of T x F x D: 64 x 64 tiles; 256 x 128 or 128 x 128 together; 256 x 256 together; 256 x 256 apart (full rounds); apart
# because the launches are long (1.6 rounds each, K = 6144)
SHAPES = [(256, 256, 1024), (1024, 768, 3072), (512, 2304, 7680), (256, 2048, 8192), (6144, 3584, 7424)]


def _codes(x, dim=None):
    amax = x.abs().max() if dim is None else x.abs().amax(dim=dim, keepdim=True)
    s = amax / 448.0
    return (x / s).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8), (float(s) if dim is None else s.reshape(-1).contiguous())


def _step(F24, kind, T, D, Fh):
    """A context and a function that runs one step of it: (Y, dX, dW1, dW2) as fresh tensors."""
    g = torch.Generator(device="cuda").manual_seed(T + D + Fh)
    rn = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
    X, W1, W2, dY = rn(T, D), rn(D, Fh) * D ** -0.5, rn(Fh, D) * Fh ** -0.5, rn(T, D)
    b1 = torch.linspace(-2, -0.5, Fh, device="cuda")
    dense, split, rowwise, fp8 = "dense" in kind, "split" in kind, "rowwise" in kind, "fp8" in kind
    flags = F24.FFN24_TRAINING | (F24.FFN24_DENSE if dense else 0) | (F24.FFN24_SPLIT if split else 0) | (F24.FFN24_ROWWISE if rowwise else 0)
    ctx = F24.Context(T, D, Fh, flags, F24.FFN24_FP8_E4M3 if fp8 else F24.FFN24_BF16)
    if split:
        ctx.set_split(256)
    fwd = ctx.ffn_fwd if dense else ctx.ffn24_fwd
    if rowwise:
        (x, sx), (w1, s1), (w2, s2) = _codes(X, 1), _codes(W1, 0), _codes(W2, 0)
        ctx.set_row_scales(sx, s1, s2)
        ops = [*_codes(dY, 1), *_codes(dY, 0), *_codes(X, 0), *_codes(W2, 1), *_codes(W1, 1)]
        bwd = ctx.ffn_bwd_rowwise if dense else ctx.ffn24_bwd_rowwise
        return ctx, lambda: (fwd(x, w1, b1, w2), *bwd(*ops)), (sx, s1, s2)
    if fp8:
        (x, sx), (w1, s1), (w2, s2), (dy, sy) = _codes(X), _codes(W1), _codes(W2), _codes(dY)
        ctx.set_scales(sx, s1, 16.0 / 448, s2)
        ctx.set_bwd_scales(sy, 32.0 / 448)
    else:
        x, w1, w2, dy = (t.bfloat16() for t in (X, W1, W2, dY))
    bwd = ctx.ffn_bwd if dense else ctx.ffn24_bwd
    return ctx, lambda: (fwd(x, w1, b1, w2), *bwd(dy)), None


@pytest.mark.parametrize("kind", ["bf16", "bf16 split", "bf16 dense", "fp8", "fp8 dense", "fp8 rowwise", "fp8 rowwise split", "fp8 rowwise dense"])
@pytest.mark.parametrize("T,D,Fh", SHAPES)
def test_profiling_gives_the_same_bits(F24, kind, T, D, Fh):
    print(f"profiling {kind} T={T} D={D} F={Fh}", flush=True)
    ctx, step, _keep = _step(F24, kind, T, D, Fh)
    plain = step()
    ctx.set_profiling(True)
    profiled = step()
    torch.cuda.synchronize()
    names = F24.KERNEL_NAMES
    times = [ctx.kernel_ms(names.index(n)) for n in (("dense_dw2", "dense_dw1") if "dense" in kind else ("dw2_sp", "dw1_sp"))]
    ctx.set_profiling(False)
    again = step()
    torch.cuda.synchronize()
    ctx.close()
    assert min(times) > 0
    assert all(bool(torch.isfinite(t.float()).all()) and float(t.float().abs().max()) > 0 for t in plain)
    for a, b, c in zip(plain, profiled, again):
        assert torch.equal(a, b) and torch.equal(a, c)
