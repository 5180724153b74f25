"""The ctypes binding without a GPU."""

import importlib.util
import types

import torch

from paper_1503_07659_amd import dgvol


def test_stream_without_torchs_raw_handle(monkeypatch):
    """Calls go to torch's current stream also where torch lacks the undocumented raw handle."""
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d: types.SimpleNamespace(cuda_stream=1000 + d))
    spec = importlib.util.spec_from_file_location(dgvol.__name__ + "_copy", dgvol.__file__)
    copy = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(copy)
    got = []
    copy._call(lambda *a: got.append(a) or dgvol.DG_OK, "entry", torch.device("cuda", 0), 5)
    assert got == [(5, 1000)]
