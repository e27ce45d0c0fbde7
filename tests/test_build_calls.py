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
