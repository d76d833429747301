"""What the build leaves where it lacks something.  (The compilers are stand-ins here: what they would write is an empty file.)"""
import os
import subprocess

import pytest

from paper_2507_19608_amd import build


@pytest.fixture
def compilers(tmp_path, monkeypatch):
    """The build into an empty directory; returns the commands that it has run.  Commands whose program is in `fails` end with an error."""
    ran, fails = [], {}

    def run(cmd, **how):
        ran.append(cmd)
        if cmd[0] in fails:
            if isinstance(fails[cmd[0]], Exception):
                raise fails[cmd[0]]
            return subprocess.CompletedProcess(cmd, 1, "", fails[cmd[0]])
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "x.hip:1:0: remark:     VGPRs Spill: 0\n" if cmd[0] == "hipcc" else "")
    monkeypatch.setattr(build, "OBJ", str(tmp_path / "_obj"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libdelta_attn.so"))
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "_marshal.so"))
    monkeypatch.setattr(build.subprocess, "run", run)
    return ran, fails


def test_everything(compilers):
    build.build()
    assert os.path.exists(build.LIB) and os.path.exists(build.MARSHAL)


@pytest.mark.parametrize("lacks", ["torch", "headers", "g++"])
def test_library_without_the_compiled_binding(compilers, monkeypatch, capsys, lacks):
    ran, fails = compilers
    open(build.MARSHAL, "w").close()                               # of an earlier build
    if lacks == "torch":
        monkeypatch.setattr(build.importlib.util, "find_spec", lambda name: None)
    else:
        fails["g++"] = "fatal error: Python.h" if lacks == "headers" else FileNotFoundError("g++")
    assert build.build() == build.LIB and os.path.exists(build.LIB)
    assert not os.path.exists(build.MARSHAL)
    said = capsys.readouterr().err
    assert "_marshal.so is not built" in said and {"headers": "Python.h"}.get(lacks, lacks) in said


def test_no_library_no_success(compilers):
    compilers[1]["hipcc"] = "error: no such kernel"
    with pytest.raises(RuntimeError, match="no such kernel"):
        build.build()
