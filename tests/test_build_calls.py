"""Building and loading the extension module of the tensor-level calls (no GPU, no compiler: the compiler is stood in for)."""
import os

import pytest

from paper_2406_07368_amd import build


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
