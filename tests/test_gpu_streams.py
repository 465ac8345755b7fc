"""Calls go to torch's current stream, found either way the binding knows."""
import pytest
import torch

from paper_2510_07651_amd import binding as obc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("raw", [True, False], ids=["raw_handle", "stream_object"])
def test_work_goes_to_the_current_stream(raw, monkeypatch):
    if raw:
        assert obc._raw_stream is not None      # (this torch has it; without it every call pays for a Stream object)
    else:
        monkeypatch.setattr(obc, "_raw_stream", None)
    scores = torch.randn(2, 4, 20000, device="cuda")
    want = scores.topk(50).indices.sort().values.int()
    side = torch.cuda.Stream()
    assert obc._stream_ptr(scores) == torch.cuda.current_stream().cuda_stream
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        assert obc._stream_ptr(scores) == side.cuda_stream
        for _ in range(20):                     # (keeps the stream busy before the copy that the call must wait for)
            late = torch.empty_like(scores).copy_(scores)
        keep = obc.obc_select(late, 50)
    side.synchronize()
    assert torch.equal(keep, want)
