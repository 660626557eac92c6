"""The stream handle that a call without a stream gets."""
import torch

from paper_2505_10938_amd import binding as B


class Current:
    cuda_stream = 1234


def test_current_stream_without_torchs_private_functions(monkeypatch):
    """A torch build that lacks the quick way to the current stream's handle takes the public one."""
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Current)
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        with monkeypatch.context() as m:
            m.delattr(torch._C, name, raising=False)
            assert B._stream(None) == 1234
    assert B._stream(Current) == 1234 and B._stream(77) == 77
