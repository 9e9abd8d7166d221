"""The binding enqueues on torch's current stream, whichever that is when a call is made."""
import pytest

pytestmark = pytest.mark.gpu


def test_calls_follow_the_current_stream():
    import torch
    import paper_2207_14696_amd.binding as b
    for s in (torch.cuda.default_stream(), torch.cuda.Stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            assert b._stream() == torch.cuda.current_stream().cuda_stream == s.cuda_stream
    assert b._stream() == torch.cuda.current_stream().cuda_stream
