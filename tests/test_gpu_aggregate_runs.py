"""aggregate_rows over runs of short lists: a lane group takes 1, 2 or 3 destinations apart from each other (by how many waves
they make), with empty and long lists at any place among them, for every number of lanes a row takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# around the 4 rows that travel together, the 4 to 64 entries a group fetches at once, and the 256 of a long list
EDGES = [0, 0, 1, 3, 4, 5, 0, 7, 8, 9, 12, 15, 16, 17, 31, 32, 33, 63, 64, 65, 257, 2, 256, 255, 0, 300, 300, 0, 1, 1025]


@pytest.mark.parametrize("waves", [3, 12_287, 12_288, 32_768])
@pytest.mark.parametrize("D,per_wave,tiles", [(3, 16, 1), (16, 16, 1), (28, 8, 1), (64, 4, 1), (100, 2, 1), (300, 1, 2), (37, 1, 1)])
def test_runs(D, per_wave, tiles, waves):
    _check(D, max(1, waves * per_wave // tiles + (waves % 2)), D + waves)


# rows that begin anywhere (their last lane shares columns with its neighbour), on both sides of one, two and three
# lists a group, and one destination more or less than a whole number of lists apart
@pytest.mark.parametrize("waves", [3, 12_287, 12_288, 32_767, 32_768])
@pytest.mark.parametrize("D,per_wave,tiles", [(4, 16, 1), (5, 16, 1), (15, 16, 1), (30, 8, 1), (101, 2, 1), (257, 1, 2)])
@pytest.mark.parametrize("more", [0, 1])
def test_row_starts(D, per_wave, tiles, waves, more):
    _check(D, -(-waves * per_wave // tiles) + more, D + waves)


# with fewer than 4 entries a list on average, two lists a group only where three are taken
@pytest.mark.parametrize("less", [0, 1])
@pytest.mark.parametrize("D,V", [(64, 12_288 * 4), (64, 32_767 * 4), (64, 32_768 * 4), (300, 6144), (300, 16_384)])
def test_few_entries(D, V, less):
    lens = np.full(V, 4)
    lens[:V // 2:2] += 3
    lens[1:V // 2:2] -= 3
    lens[7] -= less
    _check(D, V, D + V, lens)


# with fewer than two, neither (2^26 sums at most)
@pytest.mark.parametrize("D,V,less", [(64, 32_768 * 4, 0), (64, 32_768 * 4, 1), (128, 1 << 19, 1), (128, (1 << 19) + 1, 2), (300, 1 << 17, 1)])
def test_hardly_any_entries(D, V, less):
    lens = np.full(V, 2)
    lens[:V // 2:2] += 2
    lens[1:V // 2:2] -= 2
    lens[8] -= less
    _check(D, V, D + V, lens)


# 4 or 16 bytes a lane
@pytest.mark.parametrize("D,V", [(15, (1 << 18) - 1), (15, 1 << 18), (17, (1 << 17) - 1), (31, 1 << 17), (31, 70), (33, 70)])
def test_odd_widths(D, V):
    _check(D, V, D + V)


def test_narrow_odd_widths_are_no_slower():
    """Few rows of 31 columns (8 lanes of 16 bytes would share a hub's) take no longer than of 35."""
    import torch
    import paper_2207_14696_amd as bf
    V = 20_000
    rank = np.random.default_rng(0).permutation(V)
    lens = np.minimum(10_000, (3 * ((rank + 0.5) / V) ** (-1 / 1.1)).astype(np.int64) + 1)
    ptr = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)])).cuda()
    idx = torch.randint(0, V, (int(lens.sum()),), device="cuda")
    took = []
    for D in (31, 35):
        x, out = torch.randn(V, D, device="cuda"), torch.empty(V, D, device="cuda")
        best = 1e9
        for _ in range(30):
            e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e[0].record()
            bf.aggregate_rows(x, ptr, idx, out=out)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        took.append(best)
    assert took[0] < took[1], took


# Lists that together make a longer run than one list can: at the same place in every half or third of the destinations, so
# that they share a lane group, which leaves all but the first of them to others.
@pytest.mark.parametrize("waves", [12_288, 32_768])
@pytest.mark.parametrize("D,per_wave,tiles", [(20, 8, 1), (64, 4, 1), (101, 2, 1), (200, 1, 1), (300, 1, 2)])
@pytest.mark.parametrize("more", [0, 1])
def test_long_runs(D, per_wave, tiles, waves, more):
    V = -(-waves * per_wave // tiles) + more
    lens = np.random.default_rng(D + V).integers(2, 8, V)
    together = [(256, 256, 256), (256, 1, 0), (1, 255, 1), (1, 256, 0), (0, 256, 256), (128, 128, 1), (257, 10, 250), (100, 157, 99),
                (0, 0, 256), (256, 257, 256)] + [(250, 249, 248)] * 70
    for lists in (2, 3):
        step = -(-V // lists)
        for i, three in enumerate(together):
            for k in range(lists):
                if k * step + i < V:
                    lens[k * step + i + (100 if lists == 3 else 0)] = three[k]
    _check(D, V, D, lens)


def test_long_runs_are_shared():
    """Where heavy lists lie makes no difference: 200 of 250 entries at the same place in every third of the destinations, or not."""
    import torch
    import paper_2207_14696_amd as bf
    V, D = 73_728, 100
    step = V // 3
    x = torch.randn(2000, D, device="cuda")
    took = []
    for apart in (0, 1000):
        lens = torch.ones(V, dtype=torch.int64)
        for k in range(3):
            at = k * step + 1000 + k * apart
            lens[at:at + 600:3] = 250
        ptr = torch.cat([torch.zeros(1, dtype=torch.int64), lens.cumsum(0)]).cuda()
        idx = torch.randint(0, 2000, (int(lens.sum()),), device="cuda")
        out = torch.empty(V, D, device="cuda")
        best = 1e9
        for _ in range(30):
            e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e[0].record()
            bf.aggregate_rows(x, ptr, idx, out=out)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        took.append(best)
    assert took[0] < 1.5 * took[1], took


# (the index contract excludes it, the call does not look: every place read lies within the entries)
@pytest.mark.parametrize("D,V", [(100, 20), (100, 30_000), (64, 200_000), (8, 1000)])
def test_bounds_that_decrease(D, V):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(V)
    lens = rng.integers(0, 4, V)
    lens[:16] = 3                       # (what lies before any of them, 40 entries or more)
    at = rng.choice(np.arange(16, V - 1, 2), max(1, V // 50), replace=False)
    lens[at] = -2
    lens[at + 1] = 3
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    indices = rng.integers(0, 500, int(ptr.max())).astype(np.int64)
    x = torch.randn(500, D, device="cuda", generator=torch.Generator("cuda").manual_seed(D))
    out = torch.full((V, D), float("nan"), device="cuda")
    bf.aggregate_rows(x, torch.from_numpy(ptr).cuda(), torch.from_numpy(indices).cuda(), out=out, sum=True)
    want = np.zeros((V, D))
    host = x.double().cpu().numpy()
    n = np.maximum(lens, 0)
    entry = np.repeat(ptr[:-1], n) + np.concatenate([np.arange(k) for k in n])
    np.add.at(want, np.repeat(np.arange(V), n), host[indices[entry.astype(np.int64)]])
    np.testing.assert_allclose(out.cpu().numpy(), want, rtol=0, atol=6 * 2.0 ** -24 * 3 * 6)     # (|x| < 6, 3 rows)


def _check(D, V, seed, lens=None):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(seed)
    N = 5000
    if lens is None:
        lens = rng.integers(0, 10, V)                                # (4 on average, or more: as many lists a group as there can be)
        for at in (0, V // 2, max(0, V - len(EDGES))):               # the last ones end the block
            n = min(len(EDGES), V - at)
            lens[at:at + n] = rng.permutation(EDGES)[:n] if at else EDGES[:n]
    indptr = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)).cuda()
    indices = torch.from_numpy(rng.integers(0, N, int(lens.sum()))).cuda()
    x = torch.randn(N, D, device="cuda", generator=torch.Generator("cuda").manual_seed(D))
    dst = torch.repeat_interleave(torch.arange(V, device="cuda"), indptr[1:] - indptr[:-1])
    want = torch.zeros(V, D, dtype=torch.float64, device="cuda").index_add_(0, dst, x[indices].double())
    scale = torch.zeros(V, D, dtype=torch.float64, device="cuda").index_add_(0, dst, x[indices].double().abs())
    n = (indptr[1:] - indptr[:-1]).clamp(min=1)[:, None]
    # compensated sums and one division: 3 units of 2^-24 of the terms' mean size; long lists: one more for each
    # of at most 2 stretches
    for as_sum in (False, True):
        out = torch.full((V, D), float("nan"), device="cuda")
        bf.aggregate_rows(x, indptr, indices, out=out, sum=as_sum)
        per = 1 if as_sum else n
        assert torch.all((out.double() - want / per).abs() <= 6 * 2.0 ** -24 * (scale / per))
