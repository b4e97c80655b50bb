"""When a build may be skipped (the compilers are stood in for by a function that writes the output)."""
import os
import subprocess

import pytest

from paper_2505_00347_amd import build


@pytest.fixture
def tree(tmp_path, monkeypatch):
    """A source tree of its own and the list of outputs the stand-in has made; names in `fails` fail."""
    pkg = tmp_path / "pkg"
    for d in (pkg / "csrc", pkg / "lib", tmp_path / "include"):
        os.makedirs(d)
    for f in (pkg / "csrc" / "solo_py.cpp", pkg / "csrc" / "solo_api.hip", tmp_path / "include" / "solo.h"):
        f.write_text("")
        os.utime(f, (1000, 1000))
    names = {"HERE": pkg, "CSRC": pkg / "csrc", "OBJ": pkg / "_build", "LIBDIR": pkg / "lib", "LIB": pkg / "lib" / "libsolo.so",
             "NATIVE": pkg / "lib" / "native.so", "PROBE": pkg / "lib" / "probe", "EXAMPLE": pkg / "lib" / "example"}
    for name, path in names.items():
        monkeypatch.setattr(build, name, str(path))
    made, fails = [], set()

    def run(command):
        out = command[command.index("-o") + 1]
        name = os.path.basename(out).removesuffix(".new")
        if name in fails:
            raise subprocess.CalledProcessError(1, command)
        open(out, "w").close()
        made.append(name)

    monkeypatch.setattr(build.subprocess, "check_call", run)
    return names, made, fails


def test_a_failed_native_module_is_built_again(tree):
    names, made, fails = tree
    build.build()
    made.clear()
    build.build(force=False)
    assert not made                                     # everything is newer than its sources
    for f in names["CSRC"].iterdir():                   # sources change, the module's compiler fails
        os.utime(f)
    for f in (names["LIB"], names["NATIVE"]):
        os.utime(f, (2000, 2000))
    fails.add("native.so")
    with pytest.raises(subprocess.CalledProcessError):
        build.build(force=False)
    fails.clear()
    made.clear()
    build.build(force=False)
    assert "native.so" in made


def test_a_failed_link_leaves_the_old_file(tree):
    names, _, fails = tree
    build.build()
    names["LIB"].write_text("old")
    fails.add("libsolo.so")
    with pytest.raises(subprocess.CalledProcessError):
        build.build()
    assert names["LIB"].read_text() == "old"


def test_without_compiler_or_headers_no_module_is_left(tree, monkeypatch):
    names, made, _ = tree
    build.build()
    monkeypatch.setattr(build, "_native_compiler", lambda: None)
    made.clear()
    build.build()
    assert "libsolo.so" in made and "native.so" not in made and not names["NATIVE"].exists()
    made.clear()
    build.build(force=False)
    assert not made
