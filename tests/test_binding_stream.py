"""CPU test of the binding's default stream: torch's current one, through the raw
handle where torch has the function for it and through the Stream object where
it has not."""
import types

from paper_2505_06771_amd import robostep as R


def test_default_stream_with_and_without_the_raw_handle(monkeypatch):
    import torch

    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda *a: types.SimpleNamespace(cuda_stream=11))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 20 + d, raising=False)
    assert R._stream(None) == 23
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert R._stream(None) == 11
    assert R._stream(5) == 5 and R._stream(types.SimpleNamespace(cuda_stream=6)) == 6
