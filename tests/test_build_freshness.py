"""When build.py compiles a source again: what an object depends on, the compiler flags among it."""
import os

import pytest

pytest.importorskip("torch")
from paper_2411_02886_amd import build as B


@pytest.mark.parametrize("newer,again", [(None, False), ("a.hip", True), ("ts.h", True), ("tokenselect.h", True), ("build.py", True)])
def test_object_is_compiled_again_after(newer, again, tmp_path, monkeypatch):
    csrc, obj, inc = tmp_path / "csrc", tmp_path / "obj", tmp_path / "include"
    for d in (csrc, obj, inc):
        d.mkdir()
    files = {"a.hip": csrc / "a.hip", "ts.h": csrc / "ts.h", "tokenselect.h": inc / "tokenselect.h", "build.py": tmp_path / "build.py"}
    for name, f in files.items():
        f.write_text("")
        os.utime(f, (300, 300) if name == newer else (100, 100))
    (obj / "a.o").write_text("")
    os.utime(obj / "a.o", (200, 200))
    calls = []
    monkeypatch.setattr(B, "CSRC", str(csrc)); monkeypatch.setattr(B, "OBJ", str(obj)); monkeypatch.setattr(B, "ROOT", str(tmp_path))
    monkeypatch.setattr(B, "__file__", str(files["build.py"]))
    monkeypatch.setattr(B.subprocess, "check_call", calls.append)
    B._compile("a.hip", False)
    assert bool(calls) is again
