"""CPU-only tests of building and binding without the extension module that marshals torch tensors: the C library needs neither it nor PyTorch."""
import importlib.util
import os
import subprocess
import sys
import warnings

import pytest

from paper_2507_11978_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def elsewhere(tmp_path, monkeypatch):
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "CALLS", str(tmp_path / "_nt_calls.so"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libnt.so"))
    source = tmp_path / "one.cpp"
    source.write_text('extern "C" int one() { return 1; }\n')
    monkeypatch.setattr(build, "sources", lambda: [str(source)])
    return tmp_path


def test_the_library_is_built_without_pytorch(elsewhere, monkeypatch, capsys):
    real = importlib.util.find_spec
    monkeypatch.setattr(importlib.util, "find_spec", lambda name, *a: None if name == "torch" else real(name, *a))
    assert build.build(force=True) == str(elsewhere / "libnt.so") and (elsewhere / "libnt.so").exists()
    assert not (elsewhere / "_nt_calls.so").exists() and "PyTorch is not installed" in capsys.readouterr().out


def test_the_library_is_built_without_a_host_compiler_for_the_module(elsewhere, monkeypatch, capsys):
    real = subprocess.run

    def run(cmd, *args, **kwargs):
        if cmd[0] == "g++":
            raise FileNotFoundError("g++")
        return real(cmd, *args, **kwargs)
    monkeypatch.setattr(subprocess, "run", run)
    (elsewhere / "_nt_calls.so").write_bytes(b"of another torch")
    assert build.build(force=True) and (elsewhere / "libnt.so").exists()
    assert not (elsewhere / "_nt_calls.so").exists() and "through ctypes" in capsys.readouterr().out


def test_another_torch_is_built_for_again(elsewhere, monkeypatch):
    made = []

    class Result:
        returncode, stdout, stderr = 0, "", ""

    def run(cmd, *args, **kwargs):
        made.append(cmd[0])
        (elsewhere / "_nt_calls.so").write_bytes(b"")
        return Result
    monkeypatch.setattr(subprocess, "run", run)
    for version, builds in (("2.10.0", 1), ("2.10.0", 1), ("2.11.0", 2)):
        monkeypatch.setattr(build.importlib.metadata, "version", lambda name, v=version: v)
        assert build._build_calls(force=False) is None
        assert len(made) == builds


@pytest.mark.parametrize("content", [None, b"not a library"])
def test_the_binding_marshals_without_the_module(tmp_path, monkeypatch, content):
    path = tmp_path / "_nt_calls.so"
    if content is not None:
        path.write_bytes(content)
    monkeypatch.setattr(binding, "_CALLS_PATH", str(path))
    monkeypatch.setattr(binding, "_calls", None)
    with pytest.warns(RuntimeWarning, match="through ctypes"):
        assert binding._load_calls().gemm(1, 2, 3, None, None) is None
    with warnings.catch_warnings():                         # said once; the checks are the ones of the marshalling in Python
        warnings.simplefilter("error")
        import torch
        with pytest.raises(ValueError, match="GPU"):
            binding.gemm(*(torch.zeros(2, 2, dtype=torch.float16) for _ in range(3)))


def test_module_built_here_loads():
    code = "import torch, warnings; warnings.simplefilter('error'); from paper_2507_11978_amd import binding as b; print(type(b._load_calls()).__name__)"
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert out.stdout.strip() == "module", out.stderr
