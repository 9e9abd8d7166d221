"""Fused mean of few destinations, where several lane groups of a wave share a list: list lengths on both
sides of every group's share (multiples of 4 rows x 1..16 groups), the last destination alone in its tile,
with and without the caller's bound, against the oracle."""
import numpy as np
import pytest

import oracle as orc
from bifeat_inputs import FeatureSpec
from helpers import assert_close, oracle_uniform_table, scheme_of

pytestmark = pytest.mark.gpu

# rows of 16 (1 lane), 64 (4 lanes), 96 and 128 bytes (8 lanes, list entries staged), 384 and 768 (two groups, none)
@pytest.mark.parametrize("bits,D", [(1, 100), (2, 64), (4, 100), (1, 768), (8, 128), (4, 768), (8, 768)])
@pytest.mark.parametrize("V", [1, 37, 300])
def test_shared_lists(bits, D, V):
    import torch
    import paper_2207_14696_amd as bf
    spec = FeatureSpec(2500, D, 3)
    _, (mn, mx, _, _), s, codes = oracle_uniform_table(spec, bits)
    q = bf.Quantizer(scheme_of("uniform", bits), D)
    q.params_set_uniform(mn, mx)
    dcodes = torch.from_numpy(codes).cuda()
    rng = np.random.default_rng(bits * 1000 + D + V)
    edges = np.array([0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 48, 63, 64])
    deg = rng.permutation(np.resize(edges, max(V, 1)))[:V]
    deg[-1] = 64 if V == 1 else 17
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    indices = rng.integers(0, spec.N, int(indptr[-1])).astype(np.int64)
    want = orc.gather_mean(s, codes, indptr, indices)
    dptr, dind = torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda()
    for bound in (0, 64):
        q.set_option("mean_max_degree", bound)
        for ind in (dind, dind.int()):
            got = q.gather_mean(dcodes, dptr, ind)
            assert_close(got.cpu().numpy(), want, s, f"{bits} bits, D={D}, V={V}, bound {bound}, {ind.dtype}")
    assert q.poll_status()
