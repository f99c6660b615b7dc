"""The stream a call without an explicit one runs on: the current one, inside
and outside a stream context, before and after nesting."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    from paper_1203_2946_amd import cmrs
    torch.zeros(1, device="cuda")
    outer, inner = torch.cuda.Stream(), torch.cuda.Stream()
    assert cmrs._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(outer):
        assert cmrs._stream() == outer.cuda_stream
        with torch.cuda.stream(inner):
            assert cmrs._stream() == inner.cuda_stream
            assert cmrs._stream(outer) == outer.cuda_stream
        assert cmrs._stream() == outer.cuda_stream
    assert cmrs._stream() == torch.cuda.current_stream().cuda_stream
