"""The native call path is a part that may be missing: libhydra.so is built without it, and its absence is said."""
import os
import sys
import warnings

import pytest

import paper_2309_00754_amd as H
from paper_2309_00754_amd import _binding as Bd
from paper_2309_00754_amd import build as Bu


@pytest.mark.parametrize("where", ["compile", "link", "nowhere"])
def test_libhydra_is_built_without_the_native_binding(where, tmp_path, monkeypatch):
    def fail(*args):
        raise RuntimeError("no torch headers")

    def run(cmd, what):  # the link of libhydra.so
        open(cmd[cmd.index("-o") + 1], "w").close()

    monkeypatch.setattr(Bu, "BUILD", str(tmp_path / "obj"))
    monkeypatch.setattr(Bu, "LIB", str(tmp_path / "libhydra.so"))
    monkeypatch.setattr(Bu, "NATIVE", str(tmp_path / "_hydra_native.so"))
    monkeypatch.setattr(Bu, "_compile", lambda src, verbose: src + ".o")
    monkeypatch.setattr(Bu, "_run", run)
    monkeypatch.setattr(Bu, "_compile_native", fail if where == "compile" else lambda: "binding.o")
    monkeypatch.setattr(Bu, "_link_native", fail if where == "link" else lambda obj: None)
    open(Bu.NATIVE, "w").close()  # of an earlier build
    with warnings.catch_warnings(record=True) as said:
        warnings.simplefilter("always")
        assert Bu.build() == Bu.LIB
    assert os.path.exists(Bu.LIB)
    ok = where == "nowhere"
    assert os.path.exists(Bu.NATIVE) == ok
    assert ["no torch headers" in str(w.message) for w in said] == ([] if ok else [True])


@pytest.mark.parametrize("built", [True, False])
def test_a_built_binding_that_does_not_load_is_said_once(built, tmp_path, monkeypatch):
    path = tmp_path / "_hydra_native.so"
    if built:
        path.touch()
    monkeypatch.setattr(Bd, "NATIVE_PATH", str(path))
    monkeypatch.setattr(Bd, "_nat", None)
    monkeypatch.delattr(H, "_hydra_native", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2309_00754_amd._hydra_native", None)  # its import raises ImportError
    with warnings.catch_warnings(record=True) as said:
        warnings.simplefilter("always")
        assert isinstance(Bd._native(), Bd._NoNative) and isinstance(Bd._native(), Bd._NoNative)
    assert ["does not load" in str(w.message) for w in said] == [True] * built
