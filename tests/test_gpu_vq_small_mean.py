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


def _table(bf, torch, D, w, length, N, rng):
    P = D // w
    cb = rng.normal(size=(P, length, w)).astype(np.float32)
    codes = orc.pack(rng.integers(0, length, (N, P)).astype(np.uint8 if length <= 256 else np.uint16),
                     orc.vq_code_bits(length))
    q = bf.Quantizer(scheme_of("vq", 8, w, length), D)
    q.params_set_codebooks(cb)
    return q, orc.Scheme.vq(D, cb), codes, torch.from_numpy(codes).cuda()


@pytest.mark.parametrize("D,w,length", [(128, 16, 300), (64, 8, 100), (64, 4, 64)])
def test_sums_under_bounds(D, w, length):
    # from L2 (bounds up to 64) and sliced; a list beyond a bound the slices' run does not reach is
    # summed all the same
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(D + w)
    q, s, codes, dcodes = _table(bf, torch, D, w, length, 2000, rng)
    for bound, hubs in ((32, (31, 32)), (33, (33, 32)), (64, (64, 63)), (65, (65, 1)), (64, (70, 300)), (0, (500,))):
        indptr, indices = random_csr(300, 2000, 10, rng, hubs)
        want = orc.gather_mean(s, codes, indptr, indices).astype(np.float64) * np.diff(indptr)[:, None]
        scale = np.maximum(np.diff(indptr), 1)[:, None]
        q.set_option("mean_max_degree", bound)
        for sliced in (1, 2):
            q.set_option("vq_sliced", sliced)
            got = q.gather_sum(dcodes, torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda())
            assert q.poll_status()
            assert_close(got.cpu().numpy() / scale, want / scale, s, f"bound {bound} {hubs} sliced {sliced}")


def _us(torch, f):
    f()
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 5 * 1e3)
    return best


def test_a_long_list_without_a_bound_goes_through_the_slices():
    # 10 000 entries in one of 1 001 lists, nothing promised: one lane group would walk them alone
    # (2.1 ms against 0.73); the default is the sliced kernels
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(3)
    q, _, _, dcodes = _table(bf, torch, 512, 16, 2048, 20_000, rng)
    indptr, indices = random_csr(1001, 20_000, 10, rng, (10_000,))
    ptr, ind = torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda()
    out = torch.empty(1001, 512, device="cuda")
    t = {}
    for sliced in (2, 1):
        q.set_option("vq_sliced", sliced)
        t[sliced] = _us(torch, lambda: q.gather_mean(dcodes, ptr, ind, out))
    assert t[1] <= 1.5 * t[2], t


def test_workspace_of_the_sliced_mean():
    # the sliced mean takes its workspace (16 bytes and more per list entry), small bounded calls do not
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(5)
    q, s, codes, dcodes = _table(bf, torch, 768, 8, 100, 3000, rng)
    indptr, indices = random_csr(3000, 3000, 9, rng)
    ptr, ind = torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda()
    q.set_option("mean_max_degree", 9)
    want = orc.gather_mean(s, codes, indptr, indices)
    for sliced, taken in ((1, False), (2, True)):
        q.set_option("vq_sliced", sliced)
        out = torch.empty(3000, 768, device="cuda")
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        q.gather_mean(dcodes, ptr, ind, out)
        torch.cuda.synchronize()
        used = free - torch.cuda.mem_get_info()[0]
        assert (used >= 96 * len(indices)) == taken, (sliced, used)
        assert_close(out.cpu().numpy(), want, s, f"sliced {sliced}")
