"""What a fit leaves for the host: parameters read through the handle's pinned block, by a copy beyond its columns,
after a second fit, after one on another stream, and after a replayed graph of one."""
import numpy as np
import pytest

import oracle as orc
from helpers import scheme_of

pytestmark = pytest.mark.gpu


def _check(q, x, bits):
    mn, mx = orc.fit_minmax(x)
    scale, inv = orc.uniform_params(mn, mx, bits)
    for got, want in zip(q.params_get_uniform(), (mn, mx, scale, inv)):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("D", [1, 255, 768, 16384, 16385])
def test_uniform(D):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(D)
    q = bf.Quantizer(scheme_of("uniform", 4), D)
    for k in range(3):
        x = (rng.normal(size=(7, D)) * 10.0 ** k).astype(np.float32)
        t = torch.from_numpy(x).cuda()
        with torch.cuda.stream(torch.cuda.Stream() if k == 1 else torch.cuda.current_stream()):
            torch.cuda.synchronize()
            q.fit_reset()
            q.fit_update(t)
            q.fit_finalize()
        _check(q, x, 4)
        _check(q, x, 4)     # (from the host's copy)
    q.params_set_uniform(x[0], x[0] + 1)
    assert np.array_equal(q.params_get_uniform()[0], x[0])


@pytest.mark.parametrize("D", [64, 16385])
def test_uniform_replayed(D):
    """The first read after the capture is of what a replay left; what later replays leave shows in the codes."""
    import torch
    import paper_2207_14696_amd as bf
    x = np.random.default_rng(1).normal(size=(100, D)).astype(np.float32)
    t = torch.from_numpy(x).cuda()
    q = bf.Quantizer(scheme_of("uniform", 8), D)
    q.fit_reset()
    q.fit_update(t)
    q.fit_finalize()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        q.fit_reset()
        q.fit_update(t)
        q.fit_finalize()
    for k in range(3):
        y = (x * (k + 2) + k).astype(np.float32)
        t.copy_(torch.from_numpy(y))
        g.replay()
        if k == 0:
            _check(q, y, 8)
        codes = torch.zeros((100, q.row_bytes), dtype=torch.uint8, device="cuda")
        q.quantize(t, codes, 0)
        mn, mx = orc.fit_minmax(y)
        want = orc.pack(orc.uniform_encode(y, 8, mn, orc.uniform_params(mn, mx, 8)[1]), 8)
        assert np.array_equal(codes.cpu().numpy(), want)
    q.fit_reset()       # (an eager fit after them)
    q.fit_update(t)
    q.fit_finalize()
    _check(q, y, 8)


@pytest.mark.parametrize("D", [64, 16385])
def test_uniform_set_then_captured(D):
    """A fit that is captured, but not replayed, leaves the parameters that were set before it."""
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(D)
    t = torch.from_numpy(rng.normal(size=(100, D)).astype(np.float32)).cuda()
    q = bf.Quantizer(scheme_of("uniform", 8), D)
    mn = rng.normal(size=D).astype(np.float32)
    mx = mn + rng.uniform(0, 2, D).astype(np.float32)
    q.fit_update(t)
    q.fit_finalize()
    q.params_set_uniform(mn, mx)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        q.fit_reset()
        q.fit_update(t)
        q.fit_finalize()
    for got, want in zip(q.params_get_uniform(), (mn, mx, *orc.uniform_params(mn, mx, 8))):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("bits", [1, 2, 4, 8])
@pytest.mark.parametrize("clip", [0.0, 0.02])
def test_log(bits, clip):
    import torch
    import paper_2207_14696_amd as bf
    D = 300     # (more columns than the tables have entries)
    q = bf.Quantizer(scheme_of("log", bits), D)
    if clip:
        q.fit_set_log_clip(clip)
    for k in range(2):
        x = (np.random.default_rng(k).normal(size=(400, D)) * 3.0 ** k).astype(np.float32)
        t = torch.from_numpy(x).cuda()
        q.fit_reset()
        q.fit_update(t)
        while q.fit_finalize():
            q.fit_update(t)
        e_min, e_max, T, V = q.params_get_log()
        mag = np.sort(np.abs(x[x != 0]))
        lo, hi = mag[int(np.floor(clip * (mag.size - 1)))], mag[int(np.ceil((1 - clip) * (mag.size - 1)))]
        assert (e_min, e_max) == (pytest.approx(np.log2(np.float64(lo)), abs=1e-12), pytest.approx(np.log2(np.float64(hi)), abs=1e-12))
        codes = torch.zeros(400, q.row_bytes, dtype=torch.uint8, device="cuda")
        q.quantize(t, codes, 0)
        idx = torch.arange(400, device="cuda")
        rows = q.gather_dequant(codes, idx).cpu().numpy()
        level = np.searchsorted(T, np.abs(x), side="right")
        half = 1 << (bits - 1)
        want = V[np.where(x > 0, half + level, half - 1 - level)]
        assert np.array_equal(rows, want)
        # the same tables as per-column maps: means of 1- and 2-bit codes
        ptr = torch.arange(0, 401, 4, device="cuda")
        mean = q.gather_mean(codes, ptr, idx).cpu().numpy()
        np.testing.assert_allclose(mean, want.reshape(100, 4, D).astype(np.float64).mean(1), rtol=0, atol=2e-6 * np.abs(V).max())


# running states in copies: fewer workgroups than copies, more, the last columns with copies and the first without,
# extremes that only one workgroup sees
@pytest.mark.parametrize("rows,D", [(3, 5), (900, 64), (200_000, 3), (5000, 601), (3000, 8192), (300, 8196), (3, 8193)])
@pytest.mark.parametrize("half", [False, True])
def test_copies(rows, D, half):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(rows + D)
    x = rng.normal(size=(rows, D)).astype(np.float16 if half else np.float32)
    x[rng.integers(rows, size=D), np.arange(D)] = 9.0 + np.arange(D) % 50
    x[rng.integers(rows, size=D), np.arange(D)] = -9.0 - np.arange(D) % 60
    t = torch.from_numpy(x).cuda()
    cut = rows // 3
    q = bf.Quantizer(scheme_of("uniform", 8), D)
    g = bf.Quantizer(scheme_of("log", 8), D)
    for chunk in (t[:cut], t[cut:].contiguous()):
        q.fit_update(chunk)
        g.fit_update(chunk)
    q.fit_finalize()
    g.fit_finalize()
    _check(q, x.astype(np.float32), 8)
    mag = np.abs(x[x != 0].astype(np.float64))
    assert g.params_get_log()[:2] == (pytest.approx(np.log2(mag.min()), abs=1e-12), pytest.approx(np.log2(mag.max()), abs=1e-12))


@pytest.mark.parametrize("bits", [1, 2, 8])
def test_log_refit_beside_queued_gathers(bits):
    """A refit on a stream of its own leaves the tables alone that gathers queued on the default stream are to decode with."""
    import torch
    import paper_2207_14696_amd as bf
    D = 64
    x = torch.randn(500, D, device="cuda")
    q = bf.Quantizer(scheme_of("log", bits), D)
    q.params_set_log(-6.0, 1.75)
    codes = torch.zeros(500, q.row_bytes, dtype=torch.uint8, device="cuda")
    q.quantize(x, codes, 0)
    idx, ptr = torch.arange(500, device="cuda"), torch.arange(0, 501, 4, device="cuda")
    want = q.gather_dequant(codes, idx).clone(), q.gather_mean(codes, ptr, idx).clone()
    a = torch.randn(8192, 8192, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(8):      # (some ms each)
        b = a @ a
    got = q.gather_dequant(codes, idx), q.gather_mean(codes, ptr, idx)
    with torch.cuda.stream(side):
        y = x * 5
        q.fit_reset()
        q.fit_update(y)
        q.fit_finalize()
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        assert torch.equal(g, w)
    assert not torch.equal(q.gather_dequant(codes, idx), want[0])
