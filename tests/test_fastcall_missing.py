"""Without the marshalling extension every call still runs, through ctypes: where it was not built, was built for
another torch or Python, or does not load."""
import os

import pytest
import torch

from paper_2603_06664_amd import binding as B
from paper_2603_06664_amd import build

build_path = build.FASTCALL


@pytest.fixture
def fresh(monkeypatch, tmp_path):
    """The binding as after an import, with its extension in a place of its own."""
    real = B._load()
    path = str(tmp_path / "_fastcall.so")
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_fast", None)
    monkeypatch.setattr(B, "_FAST_PATH", path)
    monkeypatch.setattr(build, "FASTCALL", path)
    yield path
    monkeypatch.undo()
    B._load_fastcall(real)   # the extension's addresses are the process's: back to the library's


def _refused_call():
    """A call that the library itself refuses (no GPU needed): its own error arrives through either path."""
    t = torch.zeros((5, 3, 128), dtype=torch.bfloat16)
    with pytest.raises(B.CropeError) as e:
        B.chunk_attention(t, 5, 3, t, t, 5, [(0, 6)], 0.1, t)
    assert e.value.code == B.CROPE_ERANGE


def _unloadable(path):
    tag = build.fastcall_tag()
    with open(path, "wb") as f:
        f.write(b"no library, though for " + tag.encode())


def _other_torch(path):
    with open(build_path, "rb") as f:
        data = f.read()
    tag = build.fastcall_tag().encode()
    assert tag in data
    with open(path, "wb") as f:
        f.write(data.replace(tag, b"torch 0" + tag[7:]))


@pytest.mark.parametrize("spoil", [_unloadable, _other_torch])
def test_calls_go_through_ctypes(fresh, spoil):
    spoil(fresh)
    with pytest.warns(UserWarning, match="ctypes"):
        _refused_call()
    _refused_call()


def test_not_built_and_no_compiler(fresh, monkeypatch):
    monkeypatch.setattr(build, "_fastcall_command", lambda: ["false"])
    with pytest.warns(UserWarning, match="ctypes"):
        _refused_call()
    assert not os.path.exists(fresh)


def test_built_where_it_is_missing(fresh, monkeypatch):
    monkeypatch.setattr(build, "_fastcall_command", lambda: ["cp", build_path, fresh + ".tmp"])
    _refused_call()
    assert os.path.exists(fresh) and B._fast.append is not None
    assert type(B._fast).__name__ == "module"


def test_another_torch_makes_the_build_stale(monkeypatch):
    assert build.fastcall_current()
    monkeypatch.setattr(build, "fastcall_tag", lambda: "torch 0.1, Python 3.10")
    assert not build.fastcall_current() and build._stale()


def test_a_failed_compiler_run_leaves_no_old_extension(fresh, monkeypatch):
    with open(fresh, "wb") as f:
        f.write(b"old")
    monkeypatch.setattr(build, "_fastcall_command", lambda: ["false"])
    with pytest.warns(UserWarning, match="false failed"):
        assert not build.build_fastcall()
    assert not os.path.exists(fresh)
    monkeypatch.setattr(build, "_fastcall_command", lambda: ["no-such-compiler-here"])
    with pytest.warns(UserWarning, match="no-such-compiler-here"):
        assert not build.build_fastcall()

