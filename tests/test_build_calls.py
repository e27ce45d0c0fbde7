"""Building and loading the extension module of the tensor-level calls (no GPU, no compiler: the compiler is stood in for)."""
import os
import sys
import warnings

import pytest
import torch

from paper_2406_07368_amd import binding, build


@pytest.fixture
def place(tmp_path, monkeypatch):
    monkeypatch.setattr(build, "CALLS", str(tmp_path / "_calls.so"))
    monkeypatch.setattr(build, "CALLS_KEY", str(tmp_path / "_calls.key"))
    return tmp_path


def test_the_module_is_put_in_place_whole(place, monkeypatch):
    """While the compiler writes, and after it failed half-way, the file that another process would load is the one before; nothing is
    left behind."""
    calls = place / "_calls.so"
    calls.write_bytes(b"before")

    def compiler(then):
        def run(cmd, verbose):
            with open(cmd[cmd.index("-o") + 1], "wb") as f:
                f.write(b"half")
            assert calls.read_bytes() == b"before"
            then(cmd[cmd.index("-o") + 1])
        return run

    def fails(path):
        raise RuntimeError("out of disk")

    def ends(path):
        with open(path, "ab") as f:
            f.write(b" and half")
    monkeypatch.setattr(build, "_run", compiler(fails))
    with pytest.raises(RuntimeError):
        build.build_calls()
    assert calls.read_bytes() == b"before" and len(os.listdir(place)) == 1
    monkeypatch.setattr(build, "_run", compiler(ends))
    build.build_calls()
    assert calls.read_bytes() == b"half and half"


@pytest.mark.parametrize("missing", ["compiler", "symbol"])
def test_calls_without_the_module_take_the_general_path(place, monkeypatch, missing):
    """No compiler for a module that is not there, or one that does not load: the call itself decides (here: refuses 17 drafts), a warning
    says once why it is slower."""
    if missing == "compiler":
        def run(cmd, verbose):
            raise FileNotFoundError(cmd[0])
        monkeypatch.setattr(build, "_run", run)
    else:
        (place / "_calls.so").write_bytes(b"not a module")
        (place / "_calls.key").write_text(build.calls_key())
        monkeypatch.setitem(sys.modules, "paper_2406_07368_amd._calls", None)        # "from . import _calls" raises ImportError
        monkeypatch.delattr("paper_2406_07368_amd._calls", raising=False)
    monkeypatch.setattr(binding, "_calls", None)
    monkeypatch.setattr(binding, "_bound", None)
    q = torch.zeros(1, 1, 17, 64)
    state = (torch.zeros(1, 1, 64, 64), torch.zeros(1, 1, 64), torch.zeros(1, 1, 2, 64))

    def call():
        with pytest.raises(binding.LinattnError) as ei:
            binding.verify(q, q, q, torch.zeros(1, 64, 3), state, stream=None)
        assert ei.value.status == 2
    with pytest.warns(RuntimeWarning, match="ctypes"):
        call()
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        call()


def test_a_module_of_other_sources_or_another_torch_is_built_again(place, monkeypatch):
    def run(cmd, verbose):
        with open(cmd[cmd.index("-o") + 1], "wb") as f:
            f.write(b"module")
    monkeypatch.setattr(build, "_run", run)
    (place / "_calls.so").write_bytes(b"of unknown origin")
    assert not build.calls_current()
    build.build_calls()
    assert build.calls_current() and sorted(os.listdir(place)) == ["_calls.key", "_calls.so"]
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "0.0")
        assert not build.calls_current()
    with monkeypatch.context() as m:
        (place / "csrc").mkdir()
        with open(os.path.join(build.CSRC, "calls.cpp")) as f:
            (place / "csrc" / "calls.cpp").write_text(f.read() + "// another line\n")
        m.setattr(build, "CSRC", str(place / "csrc"))
        assert not build.calls_current()
    assert build.calls_current()
    os.remove(place / "_calls.so")
    assert not build.calls_current()


def test_the_library_does_not_wait_for_the_module(place, monkeypatch):
    """No compiler for the module: an explicit build says so, with the library in place; what loads the library asks for nothing else."""
    def run(cmd, verbose):
        if cmd[0] == "g++":
            raise FileNotFoundError("g++")
        with open(cmd[cmd.index("-o") + 1], "wb") as f:
            f.write(b"object")
    monkeypatch.setattr(build, "_run", run)
    monkeypatch.setattr(build, "LIB", str(place / "liblinattn.so"))
    monkeypatch.setattr(build, "OBJ", str(place / "_build"))
    with pytest.raises(FileNotFoundError):
        build.build()
    assert (place / "liblinattn.so").exists()
    os.remove(place / "liblinattn.so")
    assert build.build(calls=False) == str(place / "liblinattn.so") and (place / "liblinattn.so").exists()
