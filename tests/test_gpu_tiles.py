"""Every block tile of the GEMM kernel, at sizes whose shape takes it (pick_tile in tile_rule.hpp): integer products exactly, and the
fused epilogues against the oracle with the checks and bars of test_gpu_parity (bf16), or bit for bit against the same step in larger
tiles (fp8).

The tile a shape takes follows from how many tiles of each size it has; the sizes below are the smallest that take the larger tiles
with short reductions.  spmm24 is run with reduction lengths of one stage, fewer stages than the ring has slots, and odd counts beyond it.
"""
import numpy as np
import pytest
import torch

import test_gpu_parity as P
from oracle import ffn24_oracle as O
from paper_2503_16672_amd import synth

pytestmark = pytest.mark.gpu
F24 = P.F24

# up-projection tile of the shape: 64 x 64, 128 x 64, 128 x 128, 256 x 128.  The last is checked on samples of token rows and feature groups.
SHAPES = [(256, 256, 768), (512, 256, 4096), (1024, 256, 4096), (2048, 1024, 4096)]


def _samples(T, Fh):
    """Token rows and feature groups a large shape is checked on; nothing for the others, which are checked whole."""
    if T < 2048:
        return {}
    rng = np.random.default_rng(T + Fh)
    return {"rows": np.sort(rng.choice(T, 96, replace=False)), "gsel": np.sort(rng.choice(Fh // 4, 16, replace=False))}


@pytest.mark.parametrize("M,N", [(256, 256), (2048, 1024), (2048, 2048), (4096, 2048)])   # 64 x 64, 128 x 64, 128 x 128, 256 x 128
@pytest.mark.parametrize("K", [64, 128, 448, 832])
def test_spmm24_tiles_exact(F24, M, N, K):
    """Small integers: every sum is exact in fp32, and bf16 rounds it once, so the result is equal to the rounded reference."""
    print(f"spmm24 M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A = rng.integers(-3, 4, size=(M, K)).astype(np.float32)
    B = rng.integers(-3, 4, size=(N, K)).astype(np.float32)
    vals, meta = O.sparsify24(O.f32_to_bf16_bits(A))
    ref = torch.from_numpy(np.asarray(P._mm24(O.bf16_bits_to_f32(vals).astype(np.float64), meta, B.T.astype(np.float64)), np.float32)).to(torch.bfloat16)
    C = F24.spmm24(P.dev_bf16_from_words(vals), torch.from_numpy(meta).cuda(), P.to_dev_bf16(B))
    torch.cuda.synchronize()
    assert torch.equal(C.cpu(), ref)


@pytest.mark.parametrize("T,D,Fh", SHAPES)
def test_tiles_bf16(F24, T, D, Fh):
    print(f"tiles bf16 T={T} D={D} F={Fh}", flush=True)
    inp = synth.make_inputs(T, D, Fh, "per_feature", seed=T + D + Fh, with_dy=True)
    d = P._upload(inp)
    ctx = F24.Context(T, D, Fh, F24.FFN24_DEBUG_DUMP_H | F24.FFN24_TRAINING | F24.FFN24_DENSE)
    if T < 2048:
        Y = ctx.ffn24_fwd(d["X"], d["W1"], d["b1"], d["W2"])
        grads = ctx.ffn24_bwd(d["dY"])
        torch.cuda.synchronize()
        P._check_fwd24(F24, inp, ctx, d, Y)
        P._check_bwd24(F24, inp, ctx, d, grads)
    else:
        P._fwd_bwd_sampled(F24, inp, T, D, Fh, **_samples(T, Fh))
    Yd = ctx.ffn_fwd(d["X"], d["W1"], d["b1"], d["W2"])
    gd = ctx.ffn_bwd(d["dY"])
    torch.cuda.synchronize()
    f = O.ffn_fwd(inp["X"], inp["W1"], inp["b1"], inp["W2"])
    g = O.ffn_bwd(f, inp["dY"])
    errs = [O.max_rel_err(P.f64(Yd), f["Y"])] + [O.max_rel_err(P.f64(a), g[k]) for a, k in zip(gd, ("dX", "dW1", "dW2"))]
    assert max(errs) <= P.TOL_BF16
    ctx.close()


def _fp8_step(F24, q, dev, b1, rowwise, dense, ts, fs):
    """One fp8 step on the first ts tokens and fs hidden features of the inputs: (Y, dX, dW1, dW2)."""
    T, D, Fh = ts, q["X"].shape[1], fs
    ctx = F24.Context(T, D, Fh, F24.FFN24_TRAINING | (F24.FFN24_DENSE if dense else 0) | (F24.FFN24_ROWWISE if rowwise else 0), dtype=F24.FFN24_FP8_E4M3)
    X, W1, W2, dY = dev["X"][:T].contiguous(), dev["W1"][:, :Fh].contiguous(), dev["W2"][:Fh].contiguous(), dev["dY"][:T].contiguous()
    one = lambda n: torch.full((n,), 2.0 ** -6, device="cuda")
    if rowwise:
        ctx.set_row_scales(one(T), one(Fh), one(D))
    else:
        ctx.set_scales(2.0 ** -6, 2.0 ** -10, 2.0 ** -5, 2.0 ** -12)
        ctx.set_bwd_scales(2.0 ** -6, 2.0 ** -7)
    Y = (ctx.ffn_fwd if dense else ctx.ffn24_fwd)(X, W1, b1[:Fh].contiguous(), W2)
    if rowwise:
        ops = (dY, one(T), dY, one(D), X, one(D), W2, one(Fh), W1, one(D))
        g = (ctx.ffn_bwd_rowwise if dense else ctx.ffn24_bwd_rowwise)(*ops)
    else:
        g = (ctx.ffn_bwd if dense else ctx.ffn24_bwd)(dY)
    torch.cuda.synchronize()
    ctx.close()
    return (Y, *g)


@pytest.mark.parametrize("rowwise", [False, True])
@pytest.mark.parametrize("dense", [False, True])
def test_tiles_fp8_slices(F24, rowwise, dense):
    """A token's row of Y and dX depends on no other token, and a feature group's part of dW1 and dW2 on no other feature (with one scale
    per tensor, and with row-wise scales on the same slice of tokens): a step on fewer tokens or features takes smaller tiles and has to
    give the same bits, every tile summing the same k in the same order."""
    T, D, Fh = 2048, 1024, 4096
    rng = np.random.default_rng(5)
    q = {"X": rng.normal(size=(T, D)), "W1": rng.normal(size=(D, Fh)), "W2": rng.normal(size=(Fh, D)), "dY": rng.normal(size=(T, D))}
    dev = {k: torch.from_numpy((v * 64).astype(np.float32)).cuda().clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) for k, v in q.items()}
    b1 = torch.full((Fh,), -0.05, device="cuda")
    full = _fp8_step(F24, q, dev, b1, rowwise, dense, T, Fh)
    assert float(full[0].float().abs().max()) > 0 and all(bool(torch.isfinite(x.float()).all()) for x in full)
    for ts in (256, 512, 1024):
        print(f"fp8 slices rowwise={rowwise} dense={dense} tokens {ts}", flush=True)
        got = _fp8_step(F24, q, dev, b1, rowwise, dense, ts, Fh)
        assert torch.equal(got[0], full[0][:ts]) and torch.equal(got[1], full[1][:ts])
    if rowwise:
        return    # a token's scale is the maximum over all its features, so a slice of features has other scales
    for fs in (256, 768, 2048):
        print(f"fp8 slices rowwise={rowwise} dense={dense} features {fs}", flush=True)
        got = _fp8_step(F24, q, dev, b1, rowwise, dense, T, fs)
        assert torch.equal(got[2], full[2][:, :fs]) and torch.equal(got[3], full[3][:fs])


@pytest.mark.parametrize("T,D,Fh", SHAPES[1:3])
def test_tiles_split(F24, T, D, Fh):
    print(f"tiles split T={T} D={D} F={Fh}", flush=True)
    P._check_split(F24, T, D, Fh, "per_feature", T + D + Fh, 256)


@pytest.mark.parametrize("T,Fh,n_dense", [(256, 1024, 256), (2048, 2048, 512), (16384, 1280, 256)])
def test_split_partition_counts_with_ties(F24, T, Fh, n_dense):
    """The partition on counts that need one and both levels of its histogram, with every count shared by several features and with one
    count for all of them: the oracle's set, exactly (ties by feature index)."""
    g = torch.Generator().manual_seed(T + Fh)
    X = torch.randn(T, 256, generator=g).bfloat16().cuda()
    W1 = torch.randn(256, Fh // 8, generator=g).mul(1 / 16).repeat(1, 8).bfloat16().cuda()
    b1 = torch.linspace(-2, 2, Fh // 8).repeat(8).cuda()
    W2 = torch.randn(Fh, 256, generator=g).bfloat16().cuda()
    for bias in (b1, torch.full_like(b1, -1e4), torch.full_like(b1, 1e4)):
        print(f"split partition T={T} F={Fh} dense {n_dense} bias {float(bias[0])}", flush=True)
        ctx = F24.Context(T, 256, Fh, F24.FFN24_TRAINING | F24.FFN24_SPLIT)
        ctx.set_split(n_dense)
        ctx.ffn24_fwd(X, W1, bias, W2)
        ctx.ffn24_bwd(X)
        torch.cuda.synchronize()
        nnz = ctx.saved("nnz").cpu().numpy().astype(np.int64)
        assert len(np.unique(nnz)) <= Fh // 8
        dense = O.split_features(nnz, n_dense)
        assert np.array_equal(ctx.saved("feat_of_row").cpu().numpy(), np.concatenate([np.flatnonzero(~dense), np.flatnonzero(dense)]))
        ctx.close()


def test_tiles_telemetry_counts(F24):
    """Counting epilogues on the smaller tiles: the counts equal those of the tensors the GPU stored."""
    for T, D, Fh in SHAPES[:3]:
        print(f"tiles telemetry T={T} D={D} F={Fh}", flush=True)
        inp = synth.make_inputs(T, D, Fh, 0.9, seed=7 + T, with_dy=True)
        d = P._upload(inp)
        ctx = F24.Context(T, D, Fh, F24.FFN24_DEBUG_DUMP_H | F24.FFN24_TRAINING | F24.FFN24_TELEMETRY)
        ctx.ffn24_fwd(d["X"], d["W1"], d["b1"], d["W2"])
        ctx.ffn24_bwd(d["dY"])
        n = ctx.telemetry()
        assert n["nonzero"] == int((P.words_of(ctx.saved("H_dump")) != 0).sum())
        assert n["kept_tokenwise"] == int((P.words_of(ctx.saved("Hc")) != 0).sum())
        assert n["kept_featurewise"] == int((P.words_of(ctx.saved("Hc_t")) != 0).sum())
        ctx.close()


@pytest.mark.parametrize("T,Fh,with_dz", [(128, 64, True), (128, 192, True), (256, 256, False), (384, 320, True), (1152, 1088, True), (2048, 4160, False)])
def test_featurewise_rows_edges(F24, T, Fh, with_dz):
    """Row-major feature-wise re-compression at the edges of its 128 x 256 tiles (feature counts that fill a quarter, three quarters, one and a
    quarter of a tile; tile counts that are no multiple of the XCDs), signed values, with and without dZ: bit for bit against the oracle."""
    print(f"featurewise rows T={T} F={Fh} dZ={with_dz}", flush=True)
    rng = np.random.default_rng(T + Fh)
    H = rng.normal(size=(T, Fh)).astype(np.float32) * (rng.random((T, Fh)) < 0.3)
    Z = rng.normal(size=(T, Fh)).astype(np.float32)
    v, m = O.sparsify24(O.f32_to_bf16_bits(H))
    zc = O.compress_with_meta(O.f32_to_bf16_bits(Z), m)
    v_ref, m_ref = O.sparsify24(np.ascontiguousarray(O.decompress24(v, m).T))
    z_ref = O.compress_with_meta(np.ascontiguousarray(O.decompress24(zc, m).T), m_ref)
    hv, mt, zt = F24.sparsify24_featurewise(P.dev_bf16_from_words(v), torch.from_numpy(m).cuda(), P.dev_bf16_from_words(zc) if with_dz else None)
    torch.cuda.synchronize()
    assert np.array_equal(mt.cpu().numpy(), m_ref) and np.array_equal(P.words_of(hv), v_ref)
    assert (zt is None) if not with_dz else np.array_equal(P.words_of(zt), z_ref)


@pytest.mark.parametrize("R,C", [(1, 16), (2, 504), (3, 1032), (63, 520), (64, 512), (65, 1024), (130, 4096), (37, 4104), (9, 16384), (5, 16392), (16385, 16)])
def test_quantise_e4m3_edges(F24, R, C):
    """Every row width class (two, eight pieces a lane, a workgroup a row, too long for the registers), row counts at the edges of the
    column kernels' slabs (one slab, a partial one, more than 256 x 64 rows), scales from denormal to near the largest, zeros of both
    signs, infinities and NaNs: codes and scales bit for bit those of an IEEE division."""
    print(f"quantise_e4m3 edges R={R} C={C}", flush=True)
    rng = np.random.default_rng(R * 7 + C)
    x = rng.standard_normal((R, C)).astype(np.float32)
    x *= np.exp2(rng.integers(-3, 4, size=(R, 1)) * 40.0).astype(np.float32)        # 2^-120 .. 2^120
    x[rng.random((R, C)) < 0.2] = -0.0
    if R > 2:
        x[1] *= 0.0
        x[2] = np.exp2(-130.0) * rng.integers(-3, 4, size=C)
    words = O.f32_to_bf16_bits(x)
    if R > 4:
        words[3, 0] = 0x7F80
        words[4, :2] = (0xFF80, 0x7FC0)
    w = torch.from_numpy(words.view(np.int16).copy()).view(torch.bfloat16)
    xf = w.float()
    for axis in (1, 0):
        mag = torch.from_numpy((words & 0x7FFF).astype(np.int32)).amax(dim=axis)      # the largest magnitude word, NaNs above infinity
        amax = (mag << 16).view(torch.float32)
        s = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
        q = (xf / (s[:, None] if axis == 1 else s[None, :])).numpy()
        q = np.where(np.isnan(q), np.float32(-448.0), q)                               # what the saturation makes of a NaN
        ref = O.f32_to_e4m3_bits(np.clip(q, -448.0, 448.0))
        codes, scales = F24.quantise_e4m3(w.cuda(), axis)
        torch.cuda.synchronize()
        assert torch.equal(scales.cpu(), s)
        assert np.array_equal(codes.cpu().numpy(), ref)
