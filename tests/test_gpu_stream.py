"""The stream that a call without one takes: torch's current stream of the
current device, outside and inside nested stream contexts."""
import pytest

pytestmark = pytest.mark.gpu


def test_call_without_stream_takes_the_current_one():
    import torch
    from paper_2008_11520_amd import _stream
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    handle = lambda s: s.cuda_stream or None
    assert _stream(None).value == handle(torch.cuda.current_stream())
    with torch.cuda.stream(a):
        assert _stream(None).value == handle(a)
        with torch.cuda.stream(b):
            assert _stream(None).value == handle(b) and _stream(a).value == handle(a)
        assert _stream(None).value == handle(a)
    assert _stream(None).value == handle(torch.cuda.default_stream())
