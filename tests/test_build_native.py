"""The native call path is a part that may be missing: libhydra.so is built without it."""
import os
import warnings

import pytest

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
