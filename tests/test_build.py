"""What is built when: the C library by itself, and the module that calls it from Python where torch and g++ are there."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2512_19849_amd import build


@pytest.fixture
def tree(monkeypatch, tmp_path):
    """Sources in a folder of their own, and compilers that only write their output file."""
    csrc = tmp_path / "pkg" / "csrc"
    csrc.mkdir(parents=True)
    (tmp_path / "include").mkdir()
    for f in build.SOURCES + build.HEADERS + ["pycall.cpp"]:
        (csrc / f).write_text("")
    for name, value in dict(HERE=csrc.parent, CSRC=csrc, LIB=csrc.parent / "libep.so", CALL=csrc.parent / "_epcall.so",
                            CALL_SRC=csrc / "pycall.cpp").items():
        monkeypatch.setattr(build, name, str(value))
    made = []

    def run(cmd, check):
        out = cmd[cmd.index("-o") + 1]
        made.append(os.path.basename(out))
        with open(out, "w") as f:
            f.write("".join(a[len('-DEP_TORCH="'):-1].join(["torch ", "\0"]) for a in cmd if a.startswith("-DEP_TORCH=")))

    monkeypatch.setattr(build, "hipcc", lambda: "hipcc")
    monkeypatch.setattr(subprocess, "run", run)
    return made, csrc


def age(path, seconds):
    t = os.path.getmtime(path) + seconds
    os.utime(path, (t, t))


@pytest.mark.parametrize("missing", ["torch", "g++"])
def test_the_library_is_built_alone(tree, monkeypatch, missing):
    made, csrc = tree
    with open(build.CALL, "w") as f:
        f.write("of an earlier header")
    if missing == "torch":
        monkeypatch.setitem(sys.modules, "torch", None)
    else:
        monkeypatch.setattr(shutil, "which", lambda name: None)
    assert build.build_lib() == build.LIB and made[-1] == "libep.so" and not os.path.exists(build.CALL)


def test_what_is_out_of_date_is_built_again(tree, monkeypatch):
    made, csrc = tree
    torch = pytest.importorskip("torch")

    def again():
        made.clear()
        build.build_lib(force=False)
        return [m for m in made if not m.endswith(".o")]

    assert again() == ["libep.so", "_epcall.so"] and again() == []
    age(build.CALL_SRC, 100)
    assert again() == ["_epcall.so"]
    age(build.CALL_SRC, -200)
    assert again() == []
    header = os.path.join(str(csrc), "..", "..", "include", "ep.h")
    age(header, 100)
    age(build.LIB, 200)  # the library was built after the header changed, the module was not
    assert again() == ["_epcall.so"]
    age(header, -200)
    monkeypatch.setattr(torch, "__version__", "0.0")
    assert again() == ["_epcall.so"] and again() == []
    monkeypatch.setitem(sys.modules, "torch", None)  # (nothing to build it with: what is there stays for who has one)
    assert again() == [] and os.path.exists(build.CALL)
