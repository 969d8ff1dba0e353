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
