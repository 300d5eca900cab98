"""The marshalling module is an optimisation with the Python routines behind it: without it, or with one that is not of this build, the
library loads, says so and plans as before (CPU only)."""
import os
import shutil
import subprocess
import warnings

import pytest

from paper_2312_08583_amd import binding as B
from paper_2312_08583_amd import build as hip_build


@pytest.fixture
def fresh(monkeypatch):
    """The binding as before its first call, and put back afterwards."""
    B.lib()
    for name in ("_LIB", "_native_linear", "_native_group"):
        monkeypatch.setattr(B, name, getattr(B, name))
    B._LIB, B._native_linear, B._native_group = None, B._not_loaded, B._not_loaded

    def forbidden(*a, **k):
        raise AssertionError("compiles: %r" % (a,))
    monkeypatch.setattr(subprocess, "run", forbidden)
    return monkeypatch


@pytest.mark.parametrize("content", [None, b"", b"not a shared library", "library"])
def test_the_library_loads_without_the_module(fresh, tmp_path, content):
    path = str(tmp_path / "_native.so")
    if content == "library":
        shutil.copy(B.LIB_PATH, path)          # loads, but is no module
    elif content is not None:
        open(path, "wb").write(content)
    fresh.setattr(hip_build, "native_path", lambda: path)
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        plan = B.fp6_linear_plan(1, 1024, 1024)
    assert plan["workgroups"] == 32
    assert B._native_linear is B._not_loaded and B._native_group is B._not_loaded
    with warnings.catch_warnings():
        warnings.simplefilter("error")          # said once
        assert B.fp6_layout_version() == 1


def test_the_module_that_was_built_is_loaded(fresh):
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        B.lib()
    assert B._native_linear is not B._not_loaded and B._native_group is not B._not_loaded


def test_a_module_of_another_torch_or_python_is_not_taken(monkeypatch):
    import sysconfig
    import torch
    here = hip_build.native_path()
    assert here.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and os.path.dirname(here) == hip_build.HERE
    monkeypatch.setattr(torch, "__version__", "2.9.1+rocm6.4")
    assert hip_build.native_path() != here


def test_a_module_appears_whole_or_not_at_all(monkeypatch, tmp_path):
    path = tmp_path / "_native.so"
    path.write_bytes(b"the one before")
    monkeypatch.setattr(hip_build, "native_path", lambda: str(path))

    status = [1, 0]

    def link(cmd, check):
        with open(cmd[cmd.index("-o") + 1], "wb") as f:
            f.write(b"half")
            assert path.read_bytes() == b"the one before"          # what another process would import now
            f.write(b" and half")
        if status.pop(0):
            raise subprocess.CalledProcessError(1, cmd)
    monkeypatch.setattr(subprocess, "run", link)
    with pytest.raises(subprocess.CalledProcessError):
        hip_build.build_native()
    assert [p.read_bytes() for p in tmp_path.iterdir()] == [b"the one before"]
    hip_build.build_native()
    assert [p.read_bytes() for p in tmp_path.iterdir()] == [b"half and half"]
