"""Scalar codes of rows that begin anywhere: every remainder of columns by 4, rows of fewer than 4, and chunks that are
not aligned to 4 columns; the last row ends the allocation."""
import numpy as np
import pytest

import oracle as orc
from helpers import scheme_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [1, 2, 4, 8])
@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 6, 7, 9, 39, 41, 63, 130, 131, 602])
@pytest.mark.parametrize("half,shift", [(False, 0), (False, 1), (True, 1), (True, 2)])
def test_codes(bits, D, half, shift):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(D * bits)
    x = rng.normal(size=(37, D)).astype(np.float16).astype(np.float32)
    x[3, D - 1], x[5, D // 2] = np.nan, 0.0
    flat = torch.from_numpy(np.concatenate([np.zeros(shift, np.float32), x.ravel()])).cuda()
    chunk = (flat.half() if half else flat)[shift:].view(37, D)
    mn = np.full(D, -2.0, np.float32) - np.arange(D, dtype=np.float32) / 512
    mx = -mn + 0.5
    q = bf.Quantizer(scheme_of("uniform", bits), D)
    q.params_set_uniform(mn, mx)
    codes = torch.full((37, q.row_bytes), 255, dtype=torch.uint8, device="cuda")
    q.quantize(chunk, codes, 0)
    scale, inv = orc.uniform_params(mn, mx, bits)
    want = orc.pack(orc.uniform_encode(x, bits, mn, inv), bits)
    assert np.array_equal(codes.cpu().numpy(), want)
    g = bf.Quantizer(scheme_of("log", bits), D)
    g.params_set_log(-3.0, 1.0)
    codes.fill_(255)
    g.quantize(chunk, codes, 0)
    T = g.params_get_log()[2]
    H = 1 << (bits - 1)
    level = (np.abs(np.where(np.isnan(x), 0, x))[..., None] >= T).sum(-1)
    want = orc.pack(np.where(x > 0, H + level, H - 1 - level).astype(np.uint8), bits)
    assert np.array_equal(codes.cpu().numpy(), want)
