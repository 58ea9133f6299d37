"""The native one-call function is an addition: libcvx.so is built without what only that needs, and one built for another torch is
neither used nor taken for up to date."""
import os
import sys
import types

import pytest

import paper_1910_00078_amd as pkg
from paper_1910_00078_amd import build, cvx


@pytest.fixture
def runs(monkeypatch, tmp_path):
    """Commands that the build would run; their outputs appear."""
    got = []

    def run(cmd):
        got.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
    monkeypatch.setattr(build, "TORCH_LIB", str(tmp_path / "_cvx_torch.so"))
    return got, run, str(tmp_path)


@pytest.mark.parametrize("missing", ["torch", "headers", "compiler"])
def test_the_library_builds_without_torchs_prerequisites(runs, monkeypatch, missing, capsys):
    got, run, obj = runs
    if missing == "torch":
        monkeypatch.setitem(sys.modules, "torch", None)
    elif missing == "headers":
        monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": obj})
    else:
        monkeypatch.setenv("CXX", "no-such-compiler")
    build._build_torch(True, run, [], obj)
    assert not got and "missing" in capsys.readouterr().err


def test_another_torch_makes_it_stale(runs, monkeypatch):
    import torch
    got, run, obj = runs
    build._build_torch(False, run, [], obj)
    build._build_torch(False, run, [], obj)
    assert len(got) == 1 and '-DCVX_TORCH_VERSION="%s"' % torch.__version__ in got[0]
    monkeypatch.setattr(torch, "__version__", "9.9")
    build._build_torch(False, run, [], obj)
    assert len(got) == 2


@pytest.mark.parametrize("version", [None, "9.9", "ours"])
def test_one_of_another_torch_is_not_used(monkeypatch, version):
    import torch
    module = types.ModuleType("_cvx_torch")
    module.conv_fwd_fused = lambda *a: None
    if version:
        module.torch_version = str(torch.__version__) if version == "ours" else version
    monkeypatch.setattr(pkg, "_cvx_torch", module, raising=False)
    monkeypatch.setitem(sys.modules, "paper_1910_00078_amd._cvx_torch", module)
    monkeypatch.setattr(cvx, "_native", None)
    assert cvx._load_native() is (module.conv_fwd_fused if version == "ours" else False)
    assert os.path.basename(build.TORCH_LIB).startswith("_cvx_torch.cpython-")


def test_cpu_tensors_are_refused_without_the_library(monkeypatch):
    import torch

    def no_library():
        raise OSError("not built")
    monkeypatch.setattr(cvx, "lib", no_library)
    monkeypatch.setattr(cvx, "_native", None)
    with pytest.raises(ValueError, match="GPU"):
        cvx.conv_fwd_fused(torch.zeros(1, 8, 4, 4), torch.zeros(8, 8, 3, 3))
