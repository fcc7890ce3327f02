"""The current stream's handle (CPU): torch's function for the bare handle where it has one, else
the Stream object."""
import importlib.util
import sys
import types

import torch

import paper_2507_11067_amd as mms


def test_handle_without_the_private_function(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=0x70))
    spec = importlib.util.spec_from_file_location("mms_stream_probe", mms.__file__,
                                                  submodule_search_locations=mms.__path__)
    probe = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(sys.modules, "mms_stream_probe", probe)
    spec.loader.exec_module(probe)
    assert probe._stream(None).value == 0x70
    assert probe._stream(types.SimpleNamespace(cuda_stream=0x90)).value == 0x90
