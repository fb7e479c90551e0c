"""The raw stream of the call path: torch's private reader where there is one, its public interface
where there is not (CPU: the two sides of the choice; GPU: the handle of the current stream)."""
import types

import pytest

torch = pytest.importorskip("torch")

from paper_1903_06304_amd import lmfr  # noqa: E402


def test_without_the_private_reader(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=1234))
    assert lmfr._stream() == 1234


def test_with_the_private_reader(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 100 + d, raising=False)
    assert lmfr._stream() == 103


@pytest.mark.gpu
def test_current_stream():
    for s in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            assert lmfr._stream() == torch.cuda.current_stream().cuda_stream == s.cuda_stream
