"""bf16 GEMMs that read a caller's matrix with k as its slow dimension (W1, W2, X, dY where they lie): the same products in the same order as from
the re-arranged copies, so the results are equal bit for bit.  Sizes: every block tile in the up-projection, the down-projection and the weight
gradients, together, alone and with a split, and beside the feature-wise re-compression in dX (test_tile_rule.py), with one to many stages of the ring."""
from contextlib import closing

import numpy as np
import pytest
import torch

from paper_2503_16672_amd import ffn24

pytestmark = pytest.mark.gpu

SIZES = [(256, 256, 512), (256, 512, 2048), (768, 512, 2048), (1280, 768, 3072), (2048, 1024, 4096), (2048, 1280, 5120), (4096, 2048, 8192), (8192, 2048, 8192),
         (4096, 512, 1024), (2304, 1024, 1280)]


def _inputs(T, D, F):
    g = torch.Generator(device="cuda").manual_seed(T + D + F)
    new = lambda *s, scale=1.0: torch.empty(s, device="cuda").normal_(generator=g).mul_(scale).to(torch.bfloat16)
    return new(T, D), new(D, F, scale=D ** -0.5), torch.full((F,), -1.2, device="cuda"), new(F, D, scale=F ** -0.5), new(T, D)


def _equal(a, b):
    return all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(a, b, strict=True))


def _over(a, shape):
    """A matrix of `shape` and a copy of `a` that share their first bytes."""
    n = shape[0] * shape[1]
    buf = torch.zeros(max(a.numel(), n), dtype=torch.bfloat16, device="cuda")
    buf[:a.numel()] = a.reshape(-1)
    return buf[:n].view(shape), buf[:a.numel()].view(a.shape)


def _needs(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip(f"needs {gib} GiB of device memory")


def _sum_of_parts(whole, *parts):
    """The parts' sum up to the bf16 rounding of each (2^-9 of a value) and fp32 sums in another order (below 2^-12 of the 2-norm)."""
    w, p = whole.double(), [x.double() for x in parts]
    return float((w - sum(p)).norm()) <= 2.0 ** -9 * float(w.norm() + sum(x.norm() for x in p)) + 2.0 ** -12 * float(w.norm())


@pytest.mark.parametrize("T,D,F", SIZES)
@pytest.mark.parametrize("split", [0, 256])
def test_block(T, D, F, split):
    if split and (F < 1024 or (T > 2048 and F > 1280)):
        pytest.skip("a quarter of the features at most; the pair's tiles are covered by the smaller sizes")
    X, W1, b1, W2, dY = _inputs(T, D, F)
    with closing(ffn24.Context(T, D, F, ffn24.FFN24_TRAINING | ffn24.FFN24_PERMUTE | (ffn24.FFN24_SPLIT if split else 0), ffn24.FFN24_BF16)) as c:
        if split:
            c.set_split(split)
        c.set_token_permutation(np.arange(T, dtype=np.int32))       # gathers nothing, but takes the transposed copies
        c.prepare_weights(W1, W2)
        want = [c.ffn24_fwd(X, None, b1, None).clone(), *c.ffn24_bwd(dY)]
        c.set_token_permutation(None)
        for profiling in (False, True):                             # with it the weight gradients are launches of their own
            c.set_profiling(profiling)
            got = [c.ffn24_fwd(X, W1, b1, W2), *c.ffn24_bwd(dY)]
            torch.cuda.synchronize()
            assert _equal(want, got), profiling
        c.set_profiling(False)
        # an output over an input takes the copies
        Y, W2o = _over(W2, (T, D))
        assert _equal(want[:1], [c.ffn24_fwd(X, W1, b1, W2o, Y)])
        c.ffn24_fwd(X, W1, b1, W2)
        dW1, dYo = _over(dY, (D, F))
        assert _equal(want[1:], c.ffn24_bwd(dYo, out=(torch.empty_like(X), dW1, torch.empty_like(W2))))


@pytest.mark.parametrize("T,D,F", SIZES)
def test_dense(T, D, F):
    X, W1, b1, W2, dY = _inputs(T, D, F)
    with closing(ffn24.Context(T, D, F, ffn24.FFN24_TRAINING | ffn24.FFN24_DENSE, ffn24.FFN24_BF16)) as c:
        c.prepare_weights(W1, W2)
        dW1, dYo = _over(dY, (D, F))
        want = [c.ffn_fwd(X, None, b1, None).clone(), *c.ffn_bwd(dYo, out=(torch.empty_like(X), dW1, torch.empty_like(W2)))]
        for profiling in (False, True):
            c.set_profiling(profiling)
            got = [c.ffn_fwd(X, W1, b1, W2), *c.ffn_bwd(dY)]
            torch.cuda.synchronize()
            assert _equal(want, got), profiling


@pytest.mark.parametrize("T,D,F", SIZES[:5])
def test_static(T, D, F):
    X, W1, b1, W2, _ = _inputs(T, D, F)
    with closing(ffn24.Context(T, D, F, 0, ffn24.FFN24_BF16)) as c:
        c.prepare_weights(W1, W2)
        want = [c.ffn24_fwd(X, None, b1, None)]
        assert _equal(want, [ffn24.ffn24_fwd_static(X, W1, b1, W2, torch.empty_like(X))])
        Y, W2o = _over(W2, (T, D))
        assert _equal(want, [ffn24.ffn24_fwd_static(X, W1, b1, W2o, Y)])


@pytest.mark.parametrize("T,D,F", [(256, 4096, 8192), (512, 8192, 4608)])
@pytest.mark.parametrize("dense", [False, True])
def test_gradients_from_copies(T, D, F, dense):
    """Few tokens beside the gradients: dY and X are brought into panel form.  A feature's part of the gradients depends on no other feature, so a
    step on 512 features, which reads them where they lie, has the same bits."""
    X, W1, b1, W2, dY = _inputs(T, D, F)
    got = []
    for fs in (F, 512):
        with closing(ffn24.Context(T, D, fs, ffn24.FFN24_TRAINING | (ffn24.FFN24_DENSE if dense else 0), ffn24.FFN24_BF16)) as c:
            (c.ffn_fwd if dense else c.ffn24_fwd)(X, W1[:, :fs].contiguous(), b1[:fs].contiguous(), W2[:fs].contiguous())
            got.append((c.ffn_bwd if dense else c.ffn24_bwd)(dY))
    (_, dW1, dW2), (_, dW1s, dW2s) = got
    assert _equal((dW1[:, :512].contiguous(), dW2[:512]), (dW1s, dW2s))


@pytest.mark.parametrize("T,D,F", [(65536, 512, 512), (131072, 256, 512)])
@pytest.mark.parametrize("dense", [False, True])
def test_long_calls_from_copies(T, D, F, dense):
    """Many tokens beside the weights: these are brought into panel form, and (2:4) the gradients take copies of dY and X.  A token's row of Y depends on no
    other token: a forward on 1024 tokens, which reads the weights where they lie, and one with prepared weights have the same bits.  The gradients
    are the sums of those of two halves of the tokens, which read dY and X where they lie, up to the rounding of three bf16 results."""
    X, W1, b1, W2, dY = _inputs(T, D, F)

    def step(lo, hi, weights=(W1, W2)):
        with closing(ffn24.Context(hi - lo, D, F, ffn24.FFN24_TRAINING | (ffn24.FFN24_DENSE if dense else 0), ffn24.FFN24_BF16)) as c:
            if weights[0] is None:
                c.prepare_weights(W1, W2)
            Y = (c.ffn_fwd if dense else c.ffn24_fwd)(X[lo:hi], weights[0], b1, weights[1])
            return (Y, *(c.ffn_bwd if dense else c.ffn24_bwd)(dY[lo:hi]))

    full = step(0, T)
    assert _equal(full, step(0, T, (None, None)))
    assert _equal([full[0][:1024]], step(0, 1024)[:1])
    a, b = step(0, T // 2), step(T // 2, T)
    assert all(_sum_of_parts(*parts) for parts in zip(full[2:], a[2:], b[2:]))
    assert _equal([full[1]], [torch.cat([a[1], b[1]])])


def test_weights_beyond_2_gib():
    """Offsets inside a k-major operand are 32-bit: weights of 3 GiB each, both as A and as B, against the re-arranged copies, whose offsets are small."""
    T, D, F = 256, 1536, 1 << 20
    _needs(40)
    print(f"weights of 3 GiB T={T} D={D} F={F}", flush=True)
    X, W1, b1, W2, _ = _inputs(T, D, F)
    with closing(ffn24.Context(T, D, F, 0, ffn24.FFN24_BF16)) as c:
        Y = c.ffn24_fwd(X, W1, b1, W2).clone()
        c.prepare_weights(W1, W2)
        assert float(Y.float().abs().max()) > 0 and _equal([Y], [c.ffn24_fwd(X, None, b1, None)])


def test_activations_beyond_2_gib():
    """X and dY of 3 GiB: k-major in the weight gradients, and gathered by a token permutation with 32-bit offsets from their first row (the identity, against
    the rows as they stand, whose offsets are small)."""
    T, D, F = 98304, 16384, 512
    _needs(64)
    print(f"activations of 3 GiB T={T} D={D} F={F}", flush=True)
    X, W1, b1, W2, dY = _inputs(T, D, F)
    with closing(ffn24.Context(T, D, F, ffn24.FFN24_TRAINING | ffn24.FFN24_PERMUTE, ffn24.FFN24_BF16)) as c:
        got = [c.ffn24_fwd(X, W1, b1, W2).clone(), *c.ffn24_bwd(dY)]
        c.set_token_permutation(np.arange(T, dtype=np.int32))
        assert _equal(got, [c.ffn24_fwd(X, W1, b1, W2), *c.ffn24_bwd(dY)])


def test_weights_of_4_gib_take_copies():
    """Beyond 32-bit offsets the weights are re-arranged.  Y is the sum over the two halves of the features, whose weights (2 GiB) are read where they lie."""
    T, D, F = 256, 2048, 1 << 20
    _needs(48)
    print(f"weights of 4 GiB T={T} D={D} F={F}", flush=True)
    X, W1, b1, W2, _ = _inputs(T, D, F)

    def forward(lo, hi):
        with closing(ffn24.Context(T, D, hi - lo, 0, ffn24.FFN24_BF16)) as c:
            return c.ffn24_fwd(X, W1[:, lo:hi].contiguous(), b1[lo:hi].contiguous(), W2[lo:hi].contiguous())

    assert _sum_of_parts(forward(0, F), forward(0, F // 2), forward(F // 2, F))


def test_activations_of_4_gib_take_copies():
    """The same for X and dY of the weight gradients, over the two halves of the tokens; Y and dX row for row."""
    T, D, F = 1 << 20, 2048, 256
    _needs(64)
    print(f"activations of 4 GiB T={T} D={D} F={F}", flush=True)
    X, W1, b1, W2, dY = _inputs(T, D, F)

    def step(lo, hi):
        with closing(ffn24.Context(hi - lo, D, F, ffn24.FFN24_TRAINING, ffn24.FFN24_BF16)) as c:
            return c.ffn24_fwd(X[lo:hi], W1, b1, W2), *c.ffn24_bwd(dY[lo:hi])

    full, a, b = step(0, T), step(0, T // 2), step(T // 2, T)
    for i in (0, 1):
        assert _equal([full[i][:T // 2], full[i][T // 2:]], [a[i], b[i]])
    assert _sum_of_parts(full[2], a[2], b[2]) and _sum_of_parts(full[3], a[3], b[3])
