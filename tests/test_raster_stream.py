"""The stream handle of a call comes from torch's public interface where its private one is missing."""
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("device", ["cuda", "cuda:0"])
def test_public_call_serves_where_the_private_one_is_missing(monkeypatch, device):
    from paper_2412_01217_amd import raster
    seen = []

    def current_stream(d):
        seen.append(d)
        return SimpleNamespace(cuda_stream=0x1230)
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(raster, "_raw_stream", None, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    assert raster._stream(torch.device(device)) == 0x1230
    assert seen == [torch.device(device)]
