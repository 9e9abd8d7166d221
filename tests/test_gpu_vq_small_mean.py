"""Vector-code means small enough to be looked up in L2 and the same lists through the codebook slices
(option vq_sliced = 2), against the oracle: list lengths around the slices' run of 32, both index widths,
with the caller's bound kept and broken."""
import numpy as np
import pytest

import oracle as orc
from helpers import assert_close, random_csr, scheme_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,w,length", [(64, 8, 256), (128, 16, 700), (96, 4, 64), (768, 8, 100), (60, 12, 256)])
@pytest.mark.parametrize("sliced", [1, 2])
def test_small_means(D, w, length, sliced):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(D + w + length)
    N, V, P = 3000, 700, D // w
    cb = rng.normal(size=(P, length, w)).astype(np.float32)
    codes = orc.pack(rng.integers(0, length, (N, P)).astype(np.uint8 if length <= 256 else np.uint16),
                     orc.vq_code_bits(length))
    s = orc.Scheme.vq(D, cb)
    q = bf.Quantizer(scheme_of("vq", 8, w, length), D)
    q.params_set_codebooks(cb)
    q.set_option("vq_sliced", sliced)
    dcodes = torch.from_numpy(codes).cuda()
    for hubs, bound in (((31, 32, 33, 400), 0), ((31, 32), 32), ((31, 33), 32)):
        indptr, indices = random_csr(V, N, 10, rng, hubs)
        want = orc.gather_mean(s, codes, indptr, indices)
        q.set_option("mean_max_degree", bound)
        dptr = torch.from_numpy(indptr).cuda()
        broken = bound and max(hubs) > bound and w & (w - 1) == 0   # other widths promise nothing
        for ind in (torch.from_numpy(indices).cuda(), torch.from_numpy(indices).cuda().int()):
            got = q.gather_mean(dcodes, dptr, ind).cpu().numpy()
            assert q.poll_status() == (not broken)
            rows = np.arange(V) != 2 if broken else slice(None)
            assert_close(got[rows], want[rows], s, f"{hubs} bound {bound}")
            if broken:
                assert np.isnan(got[2]).all()
