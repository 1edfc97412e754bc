"""The native form of HbcsfTensor.mttkrp belongs to one torch: under another it does not load, and calls work without it."""
import importlib.util
import sys

import pytest
import torch

import paper_1904_03329_amd as pkg
from paper_1904_03329_amd import build


def _load(name):
    pkg.binding.lib()
    spec = importlib.util.spec_from_file_location(name, build.TORCH_SO)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


def test_loads_under_its_own_torch_only(monkeypatch):
    assert callable(_load("a._hbcsf_torch").mttkrp)
    monkeypatch.setattr(torch, "__version__", "0.0")
    with pytest.raises(ImportError, match="this is torch 0.0"):
        _load("b._hbcsf_torch")


@pytest.fixture
def absent(monkeypatch):
    monkeypatch.setattr(pkg, "_native_mttkrp", None)
    monkeypatch.delattr(pkg, "_hbcsf_torch", raising=False)
    monkeypatch.setitem(sys.modules, pkg.__name__ + "._hbcsf_torch", None)


def test_absence_is_a_warning(absent):
    with pytest.warns(RuntimeWarning, match="built again"):
        call = pkg._load_native()
    assert call(0, (1, 1, 1), 0, [], None) is None and pkg._native_mttkrp is call


@pytest.mark.gpu
def test_calls_work_without_it(oracle, synth, absent):
    import gpu_util as GU

    dims = (40, 30, 20)
    t = synth.tensor(dims, 3000, (0.0, 0.0, 0.0), seed=4)
    facs = synth.factors(dims, 16, seed=5)
    ht = pkg.HbcsfTensor(dims, t.inds, t.vals).to_device()
    dev = [torch.from_numpy(f).cuda() for f in facs]
    with pytest.warns(RuntimeWarning):
        first = ht.mttkrp(0, dev)
    for mode, got in enumerate([first, ht.mttkrp(1, dev), ht.mttkrp(2, dev)]):
        GU.assert_close(got.cpu().numpy(), oracle.mttkrp(dims, t.inds, t.vals, facs, mode), f"mode {mode}")
    ht.close()
