"""The native module of the per-iteration calls against the calls with an output of the caller's, which go
through ctypes: the same values, errors and streams, and arguments that it leaves to the checks in Python."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2207_14696_amd as bf
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    q = bf.Quantizer(bf.Scheme(bf.UNIFORM, 8), 24)
    q.params_set_uniform(np.zeros(24, np.float32), np.ones(24, np.float32))
    codes = torch.randint(0, 256, (500, q.row_bytes), generator=g, device="cuda", dtype=torch.uint8)
    n = torch.randint(0, 9, (64,), generator=g, device="cuda")
    indptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), n.cumsum(0)])
    indices = torch.randint(0, 500, (int(indptr[-1]),), generator=g, device="cuda")
    return bf, torch, q, codes, indptr, indices


def test_the_same_as_with_an_output(env):
    bf, torch, q, codes, indptr, indices = env
    out = torch.empty(len(indices), 24, device="cuda")
    got = q.gather_dequant(codes, indices)
    assert torch.equal(got, q.gather_dequant(codes, indices, out)) and got.dtype == torch.float32
    assert not got.requires_grad and got.is_contiguous()
    mean = torch.empty(64, 24, device="cuda")
    for lists in (indices, indices.int()):
        for call in (q.gather_mean, q.gather_sum):
            assert torch.equal(call(codes, indptr, lists), call(codes, indptr, lists, mean))
    empty = torch.empty(0, dtype=torch.int64, device="cuda")
    assert q.gather_dequant(codes, empty).shape == (0, 24)
    assert q.gather_mean(codes, indptr[:1], empty).shape == (0, 24)
    with torch.inference_mode():
        assert q.gather_dequant(codes, indices).is_inference()


def test_what_is_refused_stays_refused(env):
    bf, torch, q, codes, indptr, indices = env
    with pytest.raises(ValueError):
        q.gather_dequant(codes, indices.cpu())
    with pytest.raises(ValueError):
        q.gather_dequant(codes, indices.int())
    with pytest.raises(ValueError):
        q.gather_dequant(codes[:, ::2], indices)
    with pytest.raises(ValueError):
        q.gather_dequant(codes.float(), indices)
    with pytest.raises(ValueError):
        q.gather_mean(codes, indptr.int(), indices)
    with pytest.raises(ValueError):
        q.gather_mean(codes, indptr, indices.short())
    with pytest.raises(ValueError):
        q.gather_sum(codes, indptr[::2], indices)
    with pytest.raises(bf.BifeatError) as e:
        bf.Quantizer(bf.Scheme(bf.UNIFORM, 8), 24).gather_dequant(codes, indices)
    assert e.value.status == -2                      # not fitted
    with pytest.raises(bf.BifeatError):
        q.gather_mean(codes[:0], indptr, indices)    # an empty table
    shifted = torch.zeros(codes.numel() + 8, dtype=torch.uint8, device="cuda")[8:].view_as(codes)
    with pytest.raises(bf.BifeatError):
        q.gather_dequant(shifted, indices)           # a base that is not aligned


def test_a_destroyed_handle(env):
    bf, torch, q, codes, indptr, indices = env
    p = bf.Quantizer(bf.Scheme(bf.UNIFORM, 8), 24)
    p.params_set_uniform(np.zeros(24, np.float32), np.ones(24, np.float32))
    p.__del__()
    for call in (lambda: p.gather_dequant(codes, indices), lambda: p.gather_mean(codes, indptr, indices),
                 lambda: p.gather_sum(codes, indptr, indices.int())):
        with pytest.raises(bf.BifeatError) as e:
            call()
        assert e.value.status == bf.EINVAL


def test_a_broken_promise_is_reported_once(env):
    bf, torch, q, codes, indptr, indices = env
    p = bf.Quantizer(bf.Scheme(bf.UNIFORM, 8), 24)
    p.params_set_uniform(np.zeros(24, np.float32), np.ones(24, np.float32))
    p.set_option("mean_max_degree", 5)
    long = torch.arange(500, device="cuda").repeat(2)        # beyond what the short-list kernel holds
    p.gather_mean(codes, torch.tensor([0, 3, 1000], device="cuda"), long)
    torch.cuda.synchronize()
    with pytest.raises(bf.BifeatError):
        p.gather_mean(codes, indptr, indices)
    p.set_option("mean_max_degree", 8)
    assert torch.equal(p.gather_mean(codes, indptr, indices), q.gather_mean(codes, indptr, indices))


def test_subclasses_and_modes_take_the_python_path(env):
    bf, torch, q, codes, indptr, indices = env
    from torch.overrides import TorchFunctionMode
    want = q.gather_dequant(codes, indices)
    seen = []

    class Watch(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))
    with Watch():
        got = q.gather_dequant(codes, indices)
    assert torch.equal(got, want) and torch.empty in seen
    param = torch.nn.Parameter(codes, requires_grad=False)
    assert torch.equal(q.gather_dequant(param, indices), want)


def test_streams_and_graphs(env):
    bf, torch, q, codes, indptr, indices = env
    want = q.gather_mean(codes, indptr, indices), q.gather_dequant(codes, indices)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        got = q.gather_mean(codes, indptr, indices), q.gather_dequant(codes, indices)
    for _ in range(3):
        for t in got:
            t.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
