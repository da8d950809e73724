"""The build of the native call path (csrc/host/call.cpp): the binding works without it, so that a failure there is
reported and costs nothing else."""
import os

import pytest

from paper_2302_01425_amd import build


@pytest.fixture
def scratch(tmp_path, monkeypatch):
    """A source folder without device code and an empty library folder; hipcc is a program that does nothing."""
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    monkeypatch.setattr(build, "LIBDIR", str(tmp_path / "lib"))
    monkeypatch.setattr(build, "CALL_LIB", str(tmp_path / "lib" / "_call.so"))
    monkeypatch.setattr(build, "HIPCC", "true")
    return tmp_path


@pytest.mark.parametrize("fault", ["no compiler", "does not compile"])
def test_library_is_built_without_the_native_call(scratch, monkeypatch, capsys, fault):
    if fault == "no compiler":
        monkeypatch.setenv("CXX", str(scratch / "no-such-compiler"))
    else:
        src = scratch / "call.cpp"
        src.write_text("#error this does not compile\n")
        monkeypatch.setattr(build, "CALL_SRC", str(src))
    os.makedirs(build.LIBDIR)
    open(build.CALL_LIB, "w").close()                            # of an earlier build
    assert build.build_library(verbose=False) == build.LIB
    assert not os.path.exists(build.CALL_LIB)
    assert build.CALL_SRC in capsys.readouterr().err             # (the step that failed is named)
