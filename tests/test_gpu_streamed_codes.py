"""Large chunks: the range fit's pieces of rows (extremes planted at their edges) and codes on both sides of the
80 MB from which on they are streamed past the caches, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle as orc
from helpers import scheme_of

pytestmark = pytest.mark.gpu


# rows of a piece: 20 iterations (half precision of 768 columns: 32) of 1024 // (D / 8 or D / 4) rows (512 workgroups of 1024 threads)
@pytest.mark.parametrize("half,D,piece", [(True, 768, 320), (True, 512, 320), (False, 256, 320), (False, 100, 800)])
# (20 487: a last round of several iterations)
@pytest.mark.parametrize("over", [0, 1, 161, 20_487])
def test_range_fit(half, D, piece, over):
    import torch
    import paper_2207_14696_amd as bf
    rows = 512 * piece + over if over else 512 * piece - 1
    x = torch.rand(rows, D, device="cuda", generator=torch.Generator("cuda").manual_seed(rows))
    at = [0, piece - 1, piece, rows // 2, rows - 2, rows - 1]
    for k, r in enumerate(at):
        x[r, k::6] = 3.0 + k
        x[r, (k + 1) % 6::6] = -3.0 - k
    if half:
        x = x.half()
    q = bf.Quantizer(scheme_of("uniform", 4), D)
    q.fit_reset()
    q.fit_update(x)
    q.fit_finalize()
    mn, mx = q.params_get_uniform()[:2]
    assert np.array_equal(mn, x.amin(0).float().cpu().numpy())
    assert np.array_equal(mx, x.amax(0).float().cpu().numpy())


@pytest.mark.parametrize("kind,bits,half", [("uniform", 1, True), ("uniform", 4, False), ("uniform", 8, True), ("log", 8, True),
                                            ("log", 4, False)])
@pytest.mark.parametrize("rows", [(80 << 20) // 16, (80 << 20) // 16 + 1])
def test_codes(kind, bits, half, rows):
    import torch
    import paper_2207_14696_amd as bf
    D = 8                                                  # packed rows of 16 bytes
    x = torch.randn(rows, D, device="cuda", generator=torch.Generator("cuda").manual_seed(bits))
    if half:
        x = x.half()
    q = bf.Quantizer(scheme_of(kind, bits), D)
    host = x.float().cpu().numpy()
    if kind == "uniform":
        mn, mx = np.full(D, -3.0, np.float32), np.full(D, 3.0, np.float32)
        q.params_set_uniform(mn, mx)
        want = orc.uniform_encode(host, bits, mn, orc.uniform_params(mn, mx, bits)[1])
    else:
        q.params_set_log(-6.0, 1.75)
        want = orc.log_encode(host, bits, q.params_get_log()[2])
    codes = torch.full((rows, q.row_bytes), 0xAB, dtype=torch.uint8, device="cuda")
    q.quantize(x, codes, 0)
    assert np.array_equal(codes.cpu().numpy(), orc.pack(want, bits))
