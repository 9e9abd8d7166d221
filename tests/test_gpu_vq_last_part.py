"""Encoding where the last part has so few columns that its rows are searched by the rule: more workgroups take it."""
import numpy as np
import pytest

import oracle as orc
from helpers import scheme_of

pytestmark = pytest.mark.gpu


# one part; a few; so many that the chip holds two workgroups of each, or fewer than one; two columns of 1000 entries; 2048 entries
# (none in LDS); rows of one workgroup, of a strip and one more, of several workgroups
@pytest.mark.parametrize("D,w,length,rows", [
    (1, 8, 256, 1), (1, 8, 256, 257), (1, 8, 256, 70_001), (9, 8, 256, 3001), (33, 16, 256, 513), (129, 16, 1000, 2000), (33, 32, 256, 4001),
    (26, 8, 1000, 2500), (2401, 8, 256, 700), (6401, 8, 256, 300), (17, 16, 2048, 3000), (13, 12, 64, 1025)])
@pytest.mark.parametrize("metric,half", [("l2", False), ("l2", True), ("cosine", True)])
def test_codes(D, w, length, rows, metric, half):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(D + rows)
    x = rng.normal(size=(rows, D)).astype(np.float16).astype(np.float32)
    P = -(-D // w)
    full = rng.normal(size=(length, P * w)).astype(np.float32)
    full[:, D:] = 0
    cb = np.ascontiguousarray(full.reshape(length, P, w).transpose(1, 0, 2))
    q = bf.Quantizer(scheme_of("vq", 8, w, length, metric), D)
    q.params_set_codebooks(cb)
    codes = torch.zeros(rows, q.row_bytes, dtype=torch.uint8, device="cuda")
    t = torch.from_numpy(x).cuda()
    q.quantize(t.half() if half else t, codes, 0)
    want = orc.pack(orc.vq_assign(x, w, cb, metric=metric), orc.vq_code_bits(length))
    assert np.array_equal(codes.cpu().numpy(), want)


def test_one_column_more_is_no_dearer():
    """601 columns by 8 (the last part's rows all go by the rule) take little longer than 608."""
    import torch
    import paper_2207_14696_amd as bf
    took = []
    for D in (601, 608):
        x = torch.randn(100_000, D, device="cuda").half()
        q = bf.Quantizer(scheme_of("vq", 8, 8, 256, "l2"), D)
        q.set_option("vq_iters", 2)
        q.fit_update(x[:4096])
        q.fit_finalize()
        codes = torch.zeros(x.shape[0], q.row_bytes, dtype=torch.uint8, device="cuda")
        best = 1e9
        for _ in range(10):
            e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e[0].record()
            q.quantize(x, codes, 0)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        took.append(best)
    assert took[0] < 2 * took[1], took
