"""The native part of the binding is left out, with a warning, where it is missing or built for another torch (no GPU needed)."""
import sys
import types

import pytest

import paper_2605_29517_amd as package
from paper_2605_29517_amd import binding as M
from paper_2605_29517_amd import build as B


@pytest.fixture()
def unloaded(monkeypatch):
    monkeypatch.setattr(M, "_lib", None)
    monkeypatch.setattr(M, "_native", None)

    def native(module):
        monkeypatch.delattr(package, "_marshal", raising=False)  # (of an earlier import)
        monkeypatch.setitem(sys.modules, "paper_2605_29517_amd._marshal", module)
    return native


def test_the_build_has_one():
    from paper_2605_29517_amd import _marshal
    assert _marshal.BUILT_FOR == B.marshal_abi()


def test_missing(unloaded):
    unloaded(None)  # (an import of it raises)
    with pytest.warns(RuntimeWarning, match="missing or does not load"):
        L = M.load()
    assert M._native is None and L.maxsim_strerror(0) == b"ok" and M.load() is L


def test_built_for_another_torch(unloaded):
    def bind(*_):
        raise AssertionError("called")
    other = types.ModuleType("_marshal")
    other.BUILT_FOR, other.bind = "torch 1.0, Python 3.10", bind
    unloaded(other)
    with pytest.warns(RuntimeWarning, match="built for torch 1.0"):
        M.load()
    assert M._native is None


def test_built_before_it_said_for_what(unloaded):
    unloaded(types.ModuleType("_marshal"))
    with pytest.warns(RuntimeWarning, match="does not name"):
        M.load()
    assert M._native is None


def test_loaded_without_a_word(unloaded, recwarn):
    M.load()
    assert M._native is not None and not recwarn.list


@pytest.mark.parametrize("command", [lambda out: ["false"], lambda out: ["/nonexistent/compiler"], lambda out: 1 // 0])
def test_the_build_goes_on_without(monkeypatch, tmp_path, capsys, command):
    stale = tmp_path / "_marshal.so"
    stale.write_text("of an earlier build")
    monkeypatch.setattr(B, "MARSHAL", str(stale))
    monkeypatch.setattr(B, "marshal_command", command)
    assert B.start_marshal()() is False and not stale.exists()
    assert "does not compile here" in capsys.readouterr().err
