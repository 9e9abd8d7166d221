"""The squared distance of a training round: one value of each workgroup, summed by the kernel that makes the means."""
import numpy as np
import pytest

import oracle as orc
from helpers import scheme_of

pytestmark = pytest.mark.gpu


# workgroups: one, a few, 256 + 44, and more than 4 for each thread that sums them; the search with its sums
# (one and several sets, sets shared by workgroups) and sums from codes (2100 entries: two bytes each, 15 000 columns
# of 2 entries: plain search)
@pytest.mark.parametrize("D,w,length,rows", [
    (8, 8, 64, 64), (160, 8, 64, 5187), (2400, 8, 64, 300), (9600, 8, 32, 1024), (48, 16, 2100, 2500), (15000, 8, 2, 40)])
@pytest.mark.parametrize("metric", ["l2", "cosine"])
def test_round_distortion(D, w, length, rows, metric):
    import torch
    import paper_2207_14696_amd as bf
    x = np.random.default_rng(D + rows).normal(size=(rows, D)).astype(np.float32)
    q = bf.Quantizer(scheme_of("vq", 8, w, length, metric), D)
    q.set_option("vq_iters", 2)
    for again in range(2):      # (a second training of the handle starts from nothing)
        q.fit_reset()
        q.fit_update(torch.from_numpy(x).cuda())
        q.fit_finalize()
        got = q.vq_distortion(4)
        first = np.ascontiguousarray(x[:length].reshape(length, D // w, w).transpose(1, 0, 2))
        codes = orc.vq_assign(x, w, first, metric=metric)
        parts = x.reshape(rows, -1, w).astype(np.float64)
        want = sum(((parts[:, p] - first[p][codes[:, p]]) ** 2).sum() for p in range(D // w)) / rows
        # a distance of 8 or 16 columns in 32 bits: 10 or 18 roundings, and a lane's sum of up to 32 of them
        assert got[0] == pytest.approx(want, rel=50 * 2.0 ** -24)
        assert 0 < got[1] < got[0] or rows == length
        assert not got[2:].any()
