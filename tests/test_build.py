"""What the build makes where something that only the torch binding needs is
missing."""
from __future__ import annotations

import subprocess
import sys
import types

import pytest

from paper_2411_01738_amd import build as b


@pytest.fixture
def compilers(monkeypatch, tmp_path):
    """build() in a folder of its own, its compilers replaced by one that
    writes the output file; returns the output files in order."""
    made = []

    def run(cmd, **kw):
        out = cmd[cmd.index("-o") + 1]
        open(out, "w").close()
        made.append(out)
        return types.SimpleNamespace(returncode=0, stdout="", stderr="")

    for name in ("BUILD", "LIBRARY", "BINDING"):
        monkeypatch.setattr(b, name, str(tmp_path / name.lower()))
    monkeypatch.setattr(subprocess, "run", run)
    return made


@pytest.mark.parametrize("missing", ["torch", "g++", "Python.h"])
def test_library_without_what_the_binding_needs(compilers, monkeypatch, tmp_path, capsys, missing):
    (tmp_path / "binding").write_text("of an earlier build")
    if missing == "torch":
        for name in ("torch", "torch.utils"):
            monkeypatch.setitem(sys.modules, name, None)
    elif missing == "g++":
        monkeypatch.setattr(b.shutil, "which", lambda x: None)
    else:
        monkeypatch.setattr(b.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert b.build() == str(tmp_path / "library")
    assert (tmp_path / "library").exists() and missing in capsys.readouterr().err
    assert not (tmp_path / "binding").exists()  # nothing of another build beside the new library


def test_everything_is_built(compilers, tmp_path):
    pytest.importorskip("torch")
    b.build()
    assert (tmp_path / "library").exists() and (tmp_path / "binding").exists()
    assert len(compilers) == len(b.SOURCES) + 2
