"""Half-precision chunks, whose kernels take 8 columns per load where rows and base allow: parameters and
codes bit for bit against the oracle for column counts on both sides of that, chunks that start 8 bytes
off a 16-byte boundary, and NaN / signed zeros / infinities."""
import numpy as np
import pytest

import oracle as orc
from helpers import scheme_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [1, 2, 4, 8])
@pytest.mark.parametrize("D,rows", [(8, 1), (8, 3000), (24, 257), (100, 1000), (104, 1000), (768, 700), (12, 5000)])
@pytest.mark.parametrize("offset", [0, 4])
def test_half_chunk_codes(bits, D, rows, offset):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(D * 10 + rows + bits)
    x = (rng.normal(size=(rows, D)) * 3).astype(np.float16)
    if rows > 100:
        x[5, 0] = np.nan
        x[6, D - 1] = -0.0
        x[7, 1] = 0.0
        x[8, 2] = np.inf
    flat = torch.zeros(rows * D + 8, dtype=torch.float16, device="cuda")
    chunk = flat[offset:offset + rows * D].view(rows, D)
    chunk.copy_(torch.from_numpy(x))
    assert chunk.data_ptr() % 16 == 2 * offset
    x32 = x.astype(np.float32)

    q = bf.Quantizer(scheme_of("uniform", bits), D)
    q.fit_update(chunk)
    q.fit_finalize()
    mn, mx = orc.fit_minmax(x32)
    with np.errstate(all="ignore"):
        scale, inv = orc.uniform_params(mn, mx, bits)
        want = orc.pack(orc.uniform_encode(x32, bits, mn, inv), bits)
    for got, ref in zip(q.params_get_uniform(), (mn, mx, scale, inv)):
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))
    codes = torch.full((rows, q.row_bytes), 0xEE, dtype=torch.uint8, device="cuda")
    q.quantize(chunk, codes, 0)
    assert np.array_equal(codes.cpu().numpy(), want)

    q = bf.Quantizer(scheme_of("log", bits), D)
    q.fit_update(chunk)
    q.fit_finalize()
    e_min, e_max = orc.log_range(orc.log_fit(x32))
    T, _ = orc.log_tables(e_min, e_max, bits)
    assert q.params_get_log()[:2] == (e_min, e_max)
    q.quantize(chunk, codes, 0)
    assert np.array_equal(codes.cpu().numpy(), orc.pack(orc.log_encode(x32, bits, T), bits))


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("e_min,e_max", [(-6.0, 1.75), (-0.3, 0.4), (0.999, 1.001), (-149.0, 3.0), (-126.0, 127.9),
                                         (3.0, 3.0), (-119.5, 126.9), (100.0, 101.0)])
def test_log_levels_at_their_edges(bits, e_min, e_max):
    # every edge, the floats next to it and values all over the range, for ranges whose level follows
    # from the logarithm and for those that are searched
    import torch
    import paper_2207_14696_amd as bf
    T, _ = orc.log_tables(e_min, e_max, bits)
    rng = np.random.default_rng(bits)
    with np.errstate(all="ignore"):
        near = np.concatenate([T, np.nextafter(T, np.float32(0)), np.nextafter(T, np.float32(np.inf)),
                               np.exp2(rng.uniform(e_min - 2, e_max + 2, 4000)).astype(np.float32),
                               np.array([0.0, -0.0, np.nan, np.inf, -np.inf, 1e-45, 1e-38, 3e38], np.float32)])
    x = np.resize(np.concatenate([near, -near]), (600, 24)).astype(np.float32)
    q = bf.Quantizer(scheme_of("log", bits), 24)
    q.params_set_log(e_min, e_max)
    codes = torch.zeros((600, q.row_bytes), dtype=torch.uint8, device="cuda")
    q.quantize(torch.from_numpy(x).cuda(), codes, 0)
    want = orc.pack(orc.log_encode(x, bits, T), bits)
    bad = codes.cpu().numpy() != want
    assert not bad.any(), np.nonzero(bad.any(1))[0][:5]


@pytest.mark.parametrize("D,rows", [(8192, 37), (8200, 37), (9000, 300)])
def test_wide_half_chunks(D, rows):
    # either side of the columns whose range is merged in LDS
    import torch
    import paper_2207_14696_amd as bf
    x = (np.random.default_rng(D).normal(size=(rows, D)) * 2).astype(np.float16)
    q = bf.Quantizer(scheme_of("uniform", 4), D)
    q.fit_update(torch.from_numpy(x).cuda())
    q.fit_finalize()
    mn, mx = orc.fit_minmax(x.astype(np.float32))
    for got, ref in zip(q.params_get_uniform(), (mn, mx)):
        assert np.array_equal(got, ref)
