"""The current stream's handle where torch lacks the names of the short way: the
binding loads and takes it from torch's Stream object."""
import importlib.util
import sys
import types

import pytest
import torch


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_handle_without_the_raw_names(monkeypatch, missing):
    from paper_1203_2946_amd import cmrs
    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4711))
    spec = importlib.util.spec_from_file_location("paper_1203_2946_amd.cmrs_without", cmrs.__file__)
    m = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(sys.modules, spec.name, m)
    spec.loader.exec_module(m)
    assert m._stream() == 4711
    assert m._stream(types.SimpleNamespace(cuda_stream=7)) == 7
