"""Row-major feature-wise re-compression on both sides of the size where its tiles change (2^22 elements), at the edges of the larger ones (128
tokens x 256 features: feature counts that fill a quarter, three quarters, one and a quarter and four and a quarter tiles; tile counts that
are no multiple of the XCDs): bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import test_gpu_parity as P
from oracle import ffn24_oracle as O

pytestmark = pytest.mark.gpu
F24 = P.F24


@pytest.mark.parametrize("T,Fh,with_dz", [(2048, 2048, True), (65664, 64, True), (22016, 192, True), (13184, 320, False), (3968, 1088, True), (4224, 1024, False)])
def test_featurewise_rows_tiles(F24, T, Fh, with_dz):
    print(f"featurewise rows T={T} F={Fh} dZ={with_dz}", flush=True)
    rng = np.random.default_rng(T + Fh)
    H = rng.normal(size=(T, Fh)).astype(np.float32) * (rng.random((T, Fh)) < 0.3)
    v, m = O.sparsify24(O.f32_to_bf16_bits(H))
    zc = O.compress_with_meta(O.f32_to_bf16_bits(rng.normal(size=(T, Fh)).astype(np.float32)), m) if with_dz else None
    v_ref, m_ref = O.sparsify24(np.ascontiguousarray(O.decompress24(v, m).T))
    hv, mt, zt = F24.sparsify24_featurewise(P.dev_bf16_from_words(v), torch.from_numpy(m).cuda(), P.dev_bf16_from_words(zc) if with_dz else None)
    torch.cuda.synchronize()
    assert np.array_equal(mt.cpu().numpy(), m_ref) and np.array_equal(P.words_of(hv), v_ref)
    if with_dz:
        assert np.array_equal(P.words_of(zt), O.compress_with_meta(np.ascontiguousarray(O.decompress24(zc, m).T), m_ref))
    else:
        assert zt is None


@pytest.mark.parametrize("T,Fh", [(256, 512), (1280, 3072), (4096, 4096), (8192, 2304)])
def test_featurewise_of_a_context_equals_the_row_major_one(F24, T, Fh):
    """The context's own re-compression (panel form) against the public one, which the oracle checks above, on the tensors it started from."""
    print(f"featurewise context T={T} F={Fh}", flush=True)
    D = 256
    g = torch.Generator(device="cuda").manual_seed(T + Fh)
    new = lambda *s: torch.randn(s, device="cuda", generator=g).to(torch.bfloat16)
    ctx = F24.Context(T, D, Fh, F24.FFN24_TRAINING | F24.FFN24_TELEMETRY)
    ctx.ffn24_fwd(new(T, D), new(D, Fh), torch.full((Fh,), -16.0, device="cuda"), new(Fh, D))
    ctx.ffn24_bwd(new(T, D))
    hv, mt, zt = F24.sparsify24_featurewise(ctx.saved("Hc"), ctx.saved("meta"), ctx.saved("dZc"))
    torch.cuda.synchronize()
    assert torch.equal(ctx.saved("meta_t"), mt)
    assert torch.equal(ctx.saved("Hc_t").view(torch.int16), hv.view(torch.int16)) and torch.equal(ctx.saved("dZc_t").view(torch.int16), zt.view(torch.int16))
    assert ctx.telemetry()["kept_featurewise"] == int((hv != 0).sum())


@pytest.mark.parametrize("T,Fh", [(1792, 2048), (2048, 2048), (2304, 3072)])   # one tile of tokens a workgroup; four, from 256 workgroups on
def test_split_with_row_maxima_around_four_tiles(F24, T, Fh):
    """Every feature's scale and codes of a row-wise step with a split, bit for bit from the context's own tensors (and its weight gradients)."""
    print(f"featurewise split T={T} F={Fh}", flush=True)
    P._fp8_rowwise_split_case(F24, T, 256, Fh, "per_feature", seed=T + Fh, n_dense=512)


@pytest.mark.parametrize("T,Fh", [(256, 320), (4352, 1088)])   # 64 x 64 and 128 x 256 tiles
def test_featurewise_of_nans_and_infinities(F24, T, Fh):
    """Few words, so that most groups hold equal magnitudes: NaNs of two payloads, infinities and zeros of both signs, the neighbours of
    infinity.  The pick is by magnitude word, NaNs above infinity; ties go to the earlier token."""
    print(f"featurewise NaN T={T} F={Fh}", flush=True)
    rng = np.random.default_rng(T)
    words = np.array([0x7FC0, 0xFFC0, 0x7F81, 0xFFFF, 0x7F80, 0xFF80, 0x7F7F, 0xFF7F, 0x0000, 0x8000, 0x0001, 0x3F80], np.uint16)
    H = words[rng.integers(0, len(words), size=(T, Fh))]
    H[:, ::4] = np.where(rng.random((T, Fh // 4)) < 0.5, 0x7FC0, 0x7F80).astype(np.uint16)
    Z = rng.integers(0, 1 << 16, size=(T, Fh)).astype(np.uint16)
    v, m = O.sparsify24(H)
    zc = O.compress_with_meta(Z, m)
    v_ref, m_ref = O.sparsify24(np.ascontiguousarray(O.decompress24(v, m).T))
    z_ref = O.compress_with_meta(np.ascontiguousarray(O.decompress24(zc, m).T), m_ref)
    hv, mt, zt = F24.sparsify24_featurewise(P.dev_bf16_from_words(v), torch.from_numpy(m).cuda(), P.dev_bf16_from_words(zc))
    torch.cuda.synchronize()
    assert np.array_equal(mt.cpu().numpy(), m_ref) and np.array_equal(P.words_of(hv), v_ref) and np.array_equal(P.words_of(zt), z_ref)
