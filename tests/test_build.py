"""What the build leaves where it lacks something.  (The compilers are stand-ins here: what they would write is an empty file.)"""
import os
import subprocess
import sys
import types
import warnings

import pytest
import torch

import paper_2507_19608_amd
from paper_2507_19608_amd import binding, build


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
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / os.path.basename(build.MARSHAL)))
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
        monkeypatch.setitem(sys.modules, "torch", None)
    else:
        fails["g++"] = "fatal error: Python.h" if lacks == "headers" else FileNotFoundError("g++")
    assert build.build() == build.LIB and os.path.exists(build.LIB)
    assert not os.path.exists(build.MARSHAL)
    said = capsys.readouterr().err
    assert build.MARSHAL + " is not built" in said and {"headers": "Python.h"}.get(lacks, lacks) in said


def test_no_library_no_success(compilers):
    compilers[1]["hipcc"] = "error: no such kernel"
    with pytest.raises(RuntimeError, match="no such kernel"):
        build.build()


def test_built_again_for_another_torch(compilers, monkeypatch):
    ran, _ = compilers

    def built():
        ran.clear()
        build.build(force=False)
        return [cmd for cmd in ran if cmd[0] == "g++"]
    assert len(built()) == 1 and not built()
    monkeypatch.setattr(torch, "__version__", "1.0")
    assert any('BUILT_FOR="1.0"' in a for a in built()[0]) and not built()


def test_no_other_python_finds_it():
    assert os.path.basename(build.MARSHAL) not in ("_marshal.so", "_marshal.abi3.so")


@pytest.mark.parametrize("there", ["the right one", "another torch's", "nothing"])
def test_which_module_the_binding_takes(monkeypatch, there):
    m = types.ModuleType("_marshal")
    m.built_for = torch.__version__ if there == "the right one" else "1.0"
    monkeypatch.setattr(paper_2507_19608_amd, "_marshal", m, raising=False)
    if there == "nothing":
        monkeypatch.delattr(paper_2507_19608_amd, "_marshal")
        monkeypatch.setitem(sys.modules, "paper_2507_19608_amd._marshal", None)
    with warnings.catch_warnings(record=True) as said:
        warnings.simplefilter("always")
        assert binding._load_marshal(torch) is (m if there == "the right one" else None)
    assert len(said) == (there != "the right one")
    assert all(w.category is RuntimeWarning and "compiled marshalling is not used" in str(w.message) for w in said)
