"""The binding works without the native checks: with libvp.so alone, and where the module belongs to another PyTorch."""
import subprocess
import sys
import warnings

import pytest
import torch

import paper_2411_05288_amd.binding as B


def test_missing_module_is_not_an_error(tmp_path):
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert B._load_host(str(tmp_path / "_vphost.so")) is None
    code = ("import paper_2411_05288_amd.binding as B; B.host_path = lambda: %r; B.load_library(); "
            "assert B._HOST is None and B.vp_version() >= 100" % str(tmp_path / "_vphost.so"))
    subprocess.run([sys.executable, "-c", code], check=True, timeout=300)


def test_module_that_does_not_load(tmp_path):
    path = tmp_path / "_vphost.so"
    path.write_bytes(b"not a library")
    with pytest.warns(UserWarning, match="cannot be loaded"):
        assert B._load_host(str(path)) is None


def test_module_of_another_pytorch(monkeypatch):
    module = B._load_host(B.host_path())
    assert module is not None and module.torch_version == torch.__version__.split("+")[0]
    monkeypatch.setattr(torch, "__version__", "1.0.0")
    with pytest.warns(UserWarning, match="was built for PyTorch"):
        assert B._load_host(B.host_path()) is None
