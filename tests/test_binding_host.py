"""CPU-only: what the binding itself does between torch and the library."""
import importlib.util
import os
import types

import pytest
import torch

import ffsynth
import paper_2301_08739_amd as ff
from paper_2301_08739_amd import binding


def test_stream_without_the_short_way(monkeypatch):
    """The number of the current stream comes from a Stream object where this torch has no function for it."""
    def number():
        spec = importlib.util.spec_from_file_location("binding_of_its_own", binding.__file__)
        spec.loader.exec_module(module := importlib.util.module_from_spec(spec))
        return module._stream()
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=4711))
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert number() == 4711
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    assert number() == 103


@pytest.mark.parametrize("size", [0, 1, 100, 255, 256])
def test_tiny_workspaces_are_refused(monkeypatch, size):
    """A workspace that is smaller than what its alignment may cost has no room: the library must not be told of 2^64 bytes less some."""
    if not os.path.exists(ff.library_path()):
        pytest.skip("library not built (run __graft_entry__.build())")
    monkeypatch.setattr(binding, "_stream", lambda: None)
    ws, n = torch.empty(size, dtype=torch.uint8), 8
    layers = [ff.LayerWeights(ffsynth.layer_params(64, 128, 4, seed=1), ff.FF_F32, "cpu")]
    with pytest.raises(ff.FlatformerError, match="workspace"):
        ff.ff_fwa_block(torch.zeros(n, 3, dtype=torch.int32), ff.Geometry(1, 64, 64, 8, 8), 4, layers, ff.FF_F32, torch.zeros(n, 64),
                        workspace=ws)
    with pytest.raises(ff.FlatformerError, match="workspace"):
        ff.ff_voxelize(torch.zeros(n, 2), None, torch.zeros(n, 4), ff.Geometry(1, 64, 64, 8, 8), ff.VoxelGrid(0., 0., 1., 1.), workspace=ws)
