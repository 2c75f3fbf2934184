"""The binding's stream handle without a GPU: the given stream's, the current
stream's through torch's raw accessor, and through the public stream object
where a torch build lacks that accessor."""
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")

from paper_2212_14191_amd import tfhe


def test_given_stream():
    assert tfhe._stream(SimpleNamespace(cuda_stream=0x1230)).value == 0x1230


@pytest.mark.parametrize("has_raw", [True, False])
def test_current_stream(monkeypatch, has_raw):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=0x70))
    if has_raw:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 0x1000 + d, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert tfhe._stream().value == (0x1003 if has_raw else 0x70)
