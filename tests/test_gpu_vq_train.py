"""Codebook training in each of its forms against the oracle's rounds: the column groups of large
codebooks, codebooks on both sides of the choice between codes and the plain fused kernel, and streams
under capture that have no workspace, or not enough, to offer."""
import numpy as np
import pytest

import oracle as orc
from helpers import scheme_of

pytestmark = pytest.mark.gpu


def _train(torch, bf, x, w, length, metric, iters):
    q = bf.Quantizer(scheme_of("vq", 8, w, length, metric), x.shape[1])
    q.set_option("vq_iters", iters)
    q.fit_update(torch.from_numpy(x).cuda())
    q.fit_finalize()
    return q


# sums of 8 * length * (w + 1) bytes: 278 528 and 1.1 M for 2048 x 16 and 8000 x 16, in 144 KB a group;
# 16 384 entries leave room for one column a group (Euclidean: the directions of so many entries of two
# columns differ by 2 pi / 16 384, their cosines by 7e-8, what fp32 resolves: rounding picks the entry);
# a last part of 5 columns
@pytest.mark.parametrize("D,w,length,rows,metric", [
    (32, 16, 2048, 5000, "l2"), (32, 16, 2048, 5000, "cosine"), (21, 16, 1300, 4000, "l2"),
    (21, 16, 1300, 4000, "cosine"), (16, 16, 8000, 9000, "l2"), (16, 16, 8000, 9000, "cosine"),
    (3, 2, 16384, 17000, "l2"), (48, 48, 400, 3000, "l2"), (48, 48, 400, 3000, "cosine")])
def test_column_groups(D, w, length, rows, metric):
    import torch
    import paper_2207_14696_amd as bf
    x = np.random.default_rng(D + length).normal(size=(rows, D)).astype(np.float32)
    q = _train(torch, bf, x, w, length, metric, 2)
    cb, want = orc.vq_train(x, w, length, iters=2, metric=metric)
    # (rows between entries may change sides with the last bits of the first round's means)
    np.testing.assert_allclose(q.vq_distortion(2), want[:2], rtol=1e-4)
    assert q.vq_distortion(1)[0] == pytest.approx(want[0], rel=1e-5)
    np.testing.assert_allclose(np.abs(q.params_get_codebooks()).mean(), np.abs(cb).mean(), rtol=1e-3)


# search and sums in one kernel: workgroups of 256, 512 and 1024 threads, up to the most entries that fit and one
# more, rows that tie (searched by the rule in strips), two-byte codes, both metrics
@pytest.mark.parametrize("metric", ["l2", "cosine"])
@pytest.mark.parametrize("D,w,length,rows,kind", [
    (24, 8, 256, 3000, "normal"), (24, 8, 300, 3000, "normal"), (40, 8, 470, 3001, "normal"), (24, 8, 1000, 2100, "normal"),
    (8, 8, 1120, 2500, "normal"), (8, 8, 1121, 2500, "normal"), (32, 16, 256, 1500, "normal"), (44, 16, 500, 1500, "normal"),
    (24, 24, 150, 900, "normal"), (48, 24, 400, 1500, "normal"), (32, 32, 130, 700, "normal"), (32, 32, 290, 700, "normal"),
    (13, 13, 300, 900, "normal"), (256, 4, 16, 4100, "normal"), (12, 12, 8, 3000, "normal"), (32, 8, 8, 3000, "normal"), (24, 8, 900, 9000, "ties"), (32, 16, 300, 9000, "ties")])
def test_search_and_sums_in_one_kernel(D, w, length, rows, kind, metric):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(D + length)
    x = rng.normal(size=(rows, D)).astype(np.float32)
    if kind == "ties":
        x = rng.integers(-3, 4, size=(rows, D)).astype(np.float32)
    q = _train(torch, bf, x, w, length, metric, 1)
    cb, want = orc.vq_train(x, w, length, iters=1, metric=metric)
    if kind == "ties":      # (the oracle starts from distinct rows: its own first entries differ)
        codes = orc.vq_assign(x, w, _first_entries(x, w, length), metric=metric)
        cb, want = _one_round(x, w, length, codes)
    assert q.vq_distortion(1)[0] == pytest.approx(want[0], rel=1e-5)
    np.testing.assert_allclose(q.params_get_codebooks(), cb, rtol=2e-6, atol=1e-6)


def _first_entries(x, w, length):
    P = x.shape[1] // w
    return np.ascontiguousarray(x[:length, :P * w].reshape(length, P, w).transpose(1, 0, 2))


def _one_round(x, w, length, codes):
    cb = _first_entries(x, w, length).astype(np.float64)
    parts = x.reshape(len(x), -1, w).astype(np.float64)
    dist = 0.0
    for p in range(parts.shape[1]):
        dist += ((parts[:, p] - cb[p][codes[:, p]]) ** 2).sum()
        for e in np.unique(codes[:, p]):
            cb[p, e] = parts[codes[:, p] == e, p].mean(0)
    return cb, [dist / len(x)]


# the sums from codes, 4 columns at a time and one at a time: 1 to 16 lanes a row, column groups that are and
# are not whole fours, a last part that the table cuts short, half precision, a base that is not aligned
@pytest.mark.parametrize("D,w,length,rows,metric,half,offset", [
    (40, 8, 300, 2100, "cosine", False, 0), (36, 12, 257, 1025, "cosine", False, 0), (64, 32, 700, 1500, "l2", True, 0),
    (64, 64, 300, 1027, "l2", False, 0), (72, 24, 500, 2049, "cosine", True, 0), (40, 16, 1800, 4100, "l2", False, 0),
    (44, 16, 1800, 4100, "l2", False, 0), (40, 8, 3000, 5000, "cosine", False, 0), (40, 8, 4000, 5000, "cosine", False, 0),
    (6, 1, 64, 4100, "l2", False, 0), (12, 2, 250, 4100, "l2", False, 0), (8, 4, 30, 70, "l2", False, 0),
    (40, 8, 1500, 2000, "l2", False, 1), (38, 8, 1500, 2000, "l2", False, 0), (128, 128, 260, 600, "cosine", False, 0)])
def test_sums_from_codes(D, w, length, rows, metric, half, offset):
    import torch
    import paper_2207_14696_amd as bf
    x = np.random.default_rng(D + length).normal(size=(rows, D)).astype(np.float16 if half else np.float32)
    q = bf.Quantizer(scheme_of("vq", 8, w, length, metric), D)
    q.set_option("vq_iters", 1)
    dx = torch.zeros(rows * D + offset, dtype=torch.float16 if half else torch.float32, device="cuda")
    dx = dx[offset:].view(rows, D)
    dx.copy_(torch.from_numpy(x))
    q.fit_update(dx)
    q.fit_finalize()
    x = x.astype(np.float32)
    cb, want = orc.vq_train(x, w, length, iters=1, metric=metric)
    assert q.vq_distortion(1)[0] == pytest.approx(want[0], rel=1e-5)
    # one round: the same members in every entry, their mean rounded once (a workgroup's sums to 32 bits)
    np.testing.assert_allclose(q.params_get_codebooks(), cb, rtol=2e-6, atol=1e-6)


# A codebook's last bits: strip k of the rows belongs to set k % sets, a set's sums are rounded to 32 bits, the
# sets added in 64.  Sets of several strips and of one, a last strip that is short, several sets a workgroup (96 x
# 300 x 8, 24 x 256 x 32) and several workgroups a set (12 x 64 x 32), search and sums in one kernel and apart (64 x
# 1500 x 8, 6 x 300 x 48).  (The order of additions inside a set can move a sum over an edge between two 32-bit
# values with a chance of 1e-7.)
@pytest.mark.parametrize("P,w,length,rows,metric,strip,sets", [
    (96, 8, 256, 9000, "l2", 256, 10), (96, 8, 300, 9100, "l2", 1024, 5), (20, 16, 256, 13_000, "l2", 256, 25),
    (24, 32, 256, 33_000, "l2", 1024, 21), (40, 8, 1000, 14_000, "cosine", 1024, 12), (12, 32, 64, 4096, "cosine", 1024, 4),
    (64, 8, 1500, 9300, "l2", 1024, 8), (6, 48, 300, 5000, "l2", 1024, 5), (5, 4, 200, 700, "l2", 256, 3)])
def test_sets_of_rows(P, w, length, rows, metric, strip, sets):
    import torch
    import paper_2207_14696_amd as bf
    x = (np.random.default_rng(P + length).normal(size=(rows, P * w)) * 1.7 + 0.4).astype(np.float32)
    q = _train(torch, bf, x, w, length, metric, 1)
    want = _first_entries(x, w, length)
    codes = orc.vq_assign(x, w, want, metric=metric)
    of = np.arange(rows) // strip % sets
    for p in range(P):
        total, count = np.zeros((length, w)), np.bincount(codes[:, p], minlength=length)
        for k in range(sets):
            rows_k = np.flatnonzero(of == k)
            part = np.zeros((length, w))
            np.add.at(part, codes[rows_k, p], x[rows_k, p * w:(p + 1) * w].astype(np.float64))
            total += part.astype(np.float32)
        want[p, count > 0] = (total[count > 0] / count[count > 0, None]).astype(np.float32)
    got = q.params_get_codebooks()
    other = got != want
    assert other.sum() <= 3, f"{other.sum()} of {other.size} values differ"
    np.testing.assert_allclose(got, want, rtol=5e-7, atol=1e-7)


# rows that are near to no entry: entry 0 takes them, the Euclidean distortion is infinite (search and sums in one
# kernel, apart, the plain fused kernel)
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("P,w,length,rows,metric", [
    (3, 8, 256, 3000, "l2"), (3, 8, 300, 3000, "l2"), (2, 8, 1500, 2000, "l2"), (2, 48, 300, 900, "l2"), (3, 1, 64, 900, "l2"),
    (24, 4, 15, 900, "l2"), (16, 1, 65, 263_000, "l2"), (3, 8, 256, 3000, "cosine"), (2, 48, 300, 900, "cosine")])
def test_rows_without_a_nearest_entry(P, w, length, rows, metric, bad):
    import torch
    import paper_2207_14696_amd as bf
    x = np.random.default_rng(P + length).normal(size=(rows, P * w)).astype(np.float32)
    x[rows - 5:rows - 2, :w] = bad
    q = _train(torch, bf, x, w, length, metric, 1)
    with np.errstate(all="ignore"):
        cb, want = orc.vq_train(x, w, length, iters=1, metric=metric)
    got = q.vq_distortion(1)[0]
    assert np.isnan(got) if np.isnan(want[0]) else got == want[0] == np.inf
    np.testing.assert_array_equal(np.isnan(q.params_get_codebooks()), np.isnan(cb))


# codes or the plain fused kernel: widths 1 and 2 on both sides of 64 entries and of 2^22 rows x parts, where one and
# two columns of more entries take the latter; other widths
@pytest.mark.parametrize("P,w,length,rows", [(3, 1, 64, 5000), (3, 1, 200, 5000), (3, 1, 64, 4096), (5, 4, 31, 4097),
                                             (5, 4, 32, 4097), (130, 4, 64, 4100), (8, 2, 64, 131_200),
                                             (8, 2, 65, 131_200), (4, 5, 40, 700), (1, 64, 30, 900),
                                             (64, 1, 65, 65_535), (64, 1, 65, 65_536), (64, 1, 64, 65_536),
                                             (128, 2, 64, 32_768), (128, 2, 65, 32_768), (128, 2, 65, 32_767)])
def test_small_codebooks(P, w, length, rows):
    import torch
    import paper_2207_14696_amd as bf
    x = np.random.default_rng(P * w + length).normal(size=(rows, P * w)).astype(np.float32)
    q = _train(torch, bf, x, w, length, "l2", 2)
    _, want = orc.vq_train(x, w, length, iters=2)
    np.testing.assert_allclose(q.vq_distortion(2), want[:2], rtol=2e-5)


@pytest.mark.parametrize("P,w,length,metric,reserve", [
    (4, 16, 256, "l2", 0), (4, 16, 256, "cosine", 0), (4, 8, 700, "l2", 0),  # search and sums, no room: one set of sums
    (4, 8, 32, "l2", 0), (4, 8, 32, "l2", 20_000), (2, 5, 40, "l2", 20_000),  # the plain fused kernel
    (2, 16, 700, "cosine", 20_000)])  # room for the codes only: one set of sums
def test_training_under_capture(P, w, length, metric, reserve):
    import torch
    import paper_2207_14696_amd as bf
    rng = np.random.default_rng(length)
    x = rng.normal(size=(20_000, P * w)).astype(np.float32)
    dx = torch.from_numpy(x).cuda()
    eager = bf.Quantizer(scheme_of("vq", 8, w, length, metric), P * w)
    eager.fit_update(dx)
    want = eager.vq_distortion(10)
    q = bf.Quantizer(scheme_of("vq", 8, w, length, metric), P * w)
    q.fit_reset()
    if reserve:
        q.reserve(reserve)
    g, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(g, stream=stream):
        q.fit_update(dx)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        got = q.vq_distortion(10)
        assert got[0] == pytest.approx(want[0], rel=1e-5)
        np.testing.assert_allclose(got, want, rtol=2e-3)   # ten rounds from sums in another order
        dx.mul_(1.0)                                       # the program's own work between replays
    eager.fit_update(dx)


# a codebook that goes through codes for up to 2^18 rows x parts (513 parts: 511 rows) and cannot do without them: a larger
# update, which needs none, leaves room for them all the same
def test_a_smaller_update_under_capture_after_a_larger_one():
    import torch
    import paper_2207_14696_amd as bf
    P, w, length = 513, 4, 16
    x = torch.from_numpy(np.random.default_rng(5).normal(size=(600, P * w)).astype(np.float32)).cuda()
    q, eager = (bf.Quantizer(scheme_of("vq", 8, w, length, "cosine"), P * w) for _ in range(2))
    q.fit_update(x)
    q.fit_reset()
    small = x[:511].contiguous()
    g, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(g, stream=stream):
        q.fit_update(small)
    eager.fit_update(small)
    want = eager.vq_distortion(10)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_allclose(q.vq_distortion(10), want, rtol=1e-5)
        small.mul_(1.0)


def _us(torch, f):
    f()
    best = 1e9
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("P,w,length,reserve", [(8, 16, 256, 0), (12, 8, 32, 65_536), (8, 16, 1024, 65_536)])
def test_training_under_capture_fills_the_chip(P, w, length, reserve):
    # search and sums in one kernel, twice, and the sums from codes, each with room for one set: 0.9 to 1.0 times an eager
    # call's time; with a workgroup per part it was 6 to 13 times
    import torch
    import paper_2207_14696_amd as bf
    x = torch.randn(65_536, P * w, device="cuda")
    q = bf.Quantizer(scheme_of("vq", 8, w, length), P * w)
    q.fit_reset()
    if reserve:
        q.reserve(reserve)
    g, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(g, stream=stream):
        q.fit_update(x)
    captured = _us(torch, g.replay)
    eager = bf.Quantizer(scheme_of("vq", 8, w, length), P * w)

    def call():
        eager.fit_reset()
        eager.fit_update(x)
    t = _us(torch, call)
    assert captured <= 3 * t, (captured, t)
