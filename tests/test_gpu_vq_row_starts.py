"""Sample rows that begin anywhere: encode and training where rows, or the chunk, are not aligned to 4 columns, and a
last part with 1 to 3 columns more than whole fours."""
import numpy as np
import pytest

import oracle as orc
from helpers import scheme_of

pytestmark = pytest.mark.gpu


def _chunk(torch, x, half, shift):
    """x on the GPU, `shift` elements into an allocation; the last row ends it."""
    flat = torch.from_numpy(np.concatenate([np.zeros(shift, x.dtype), x.ravel()])).cuda()
    return (flat.half() if half else flat)[shift:].view(x.shape)


# the search on the matrix cores (widths of up to 8, 16, 24, 32 columns) and the plain one (few entries)
@pytest.mark.parametrize("w,length", [(4, 64), (8, 32), (12, 64), (16, 64), (20, 40), (32, 40), (8, 2), (16, 2), (5, 64)])
@pytest.mark.parametrize("tail", [0, 1, 2, 3])
@pytest.mark.parametrize("half,shift", [(False, 0), (False, 1), (True, 0), (True, 1), (True, 2)])
def test_encode(w, length, tail, half, shift):
    import torch
    import paper_2207_14696_amd as bf
    D = 2 * w + max(0, w - 4 + tail) if tail else 2 * w
    rng = np.random.default_rng(w * 10 + tail)
    x = rng.normal(size=(333, D)).astype(np.float16).astype(np.float32)
    P = -(-D // w)
    full = rng.normal(size=(length, P * w)).astype(np.float32)
    full[:, D:] = 0
    cb = np.ascontiguousarray(full.reshape(length, P, w).transpose(1, 0, 2))
    for metric in ("l2", "cosine"):
        q = bf.Quantizer(scheme_of("vq", 8, w, length, metric), D)
        q.params_set_codebooks(cb)
        codes = torch.zeros(333, q.row_bytes, dtype=torch.uint8, device="cuda")
        q.quantize(_chunk(torch, x, half, shift), codes, 0)
        want = orc.vq_assign(x, w, cb, metric=metric)
        assert np.array_equal(codes.cpu().numpy()[:, :P], want)


# sums in the search's kernel, and from codes (2100 entries, two bytes)
@pytest.mark.parametrize("D,w,length,rows", [(43, 16, 64, 700), (21, 8, 40, 700), (47, 16, 2100, 2400), (30, 12, 300, 700)])
@pytest.mark.parametrize("half,shift", [(False, 1), (True, 1)])
def test_train(D, w, length, rows, half, shift):
    import torch
    import paper_2207_14696_amd as bf
    x = np.random.default_rng(D).normal(size=(rows, D)).astype(np.float16).astype(np.float32)
    q = bf.Quantizer(scheme_of("vq", 8, w, length, "l2"), D)
    q.set_option("vq_iters", 1)
    q.fit_update(_chunk(torch, x, half, shift))
    q.fit_finalize()
    cb, want = orc.vq_train(x, w, length, iters=1, metric="l2")
    assert q.vq_distortion(1)[0] == pytest.approx(want[0], rel=1e-5)
    # a mean is a 64-bit sum rounded to 32 bits set by set, then divided: 2^-23 of the sum's size
    np.testing.assert_allclose(q.params_get_codebooks(), cb, rtol=2e-6, atol=1e-6)
