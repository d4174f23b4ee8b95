"""The build: the C library needs neither torch nor Python headers, so a
marshalling module that cannot be built still leaves it installed, and the
error says what is missing."""
import importlib.util
import os

import pytest

from paper_2607_16673_amd import build as hip_build


@pytest.fixture
def scratch(tmp_path, monkeypatch):
    """One source of the library, built under tmp_path."""
    for name, path in (("BUILD", "obj"), ("LIB", "libsla.so"), ("NATIVE", "_native.so")):
        monkeypatch.setattr(hip_build, name, str(tmp_path / path))
    monkeypatch.setattr(hip_build, "SOURCES", [("verify_tile_dispatch.cpp", "dispatch", [])])
    return tmp_path


@pytest.mark.parametrize("missing", ["torch", "g++", "headers"])
def test_library_is_installed_without_the_module(scratch, monkeypatch, missing):
    if missing == "torch":
        find = importlib.util.find_spec
        monkeypatch.setattr(importlib.util, "find_spec", lambda name, *a: None if name == "torch" else find(name, *a))
    elif missing == "g++":
        run = hip_build.subprocess.run

        def no_gxx(cmd, **k):
            if cmd[0] == "g++":
                raise FileNotFoundError(cmd[0])
            return run(cmd, **k)

        monkeypatch.setattr(hip_build.subprocess, "run", no_gxx)
    else:
        monkeypatch.setattr(hip_build.sysconfig, "get_paths", lambda: {"include": str(scratch)})
        monkeypatch.setattr(hip_build, "_torch_dir", lambda: str(scratch), raising=False)
    what = {"torch": "torch is not installed", "g++": r"g\+\+ is not installed", "headers": "failed for torch_binding.cpp"}
    with pytest.raises(RuntimeError, match=what[missing]):
        hip_build.build()
    assert os.path.exists(hip_build.LIB)
    assert not os.path.exists(hip_build.NATIVE)
