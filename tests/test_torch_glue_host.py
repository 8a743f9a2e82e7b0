"""torch_glue without the undocumented torch function that gives a stream's handle."""
import importlib.util
import os
import types

import torch

import paper_2510_08318_amd as package


def test_stream_handle_without_torchs_own_function(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    spec = importlib.util.spec_from_file_location(package.__name__ + ".glue_copy", os.path.join(os.path.dirname(package.__file__), "torch_glue.py"))
    glue = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(glue)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: types.SimpleNamespace(cuda_stream=100 + device))
    assert glue._current_stream() == 103
