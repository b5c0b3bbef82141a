"""The current stream without torch's private calls, which other builds of it may not have."""
import torch


def test_public_lookup(monkeypatch):
    from paper_2602_08642_amd import ops
    class S:
        cuda_stream = 4711
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: S)
    for name in ("_raw_stream", "_current_device"):
        with monkeypatch.context() as m:
            m.setattr(ops, name, None)
            assert ops._stream() == 4711
