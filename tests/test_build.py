"""The build script: what it needs, without compiling anything."""
import importlib.util
import subprocess

import pytest

from paper_2412_04964_amd import build


@pytest.fixture
def commands(monkeypatch, tmp_path):
    """Runs no command; collects the libraries that would have been linked, and the failures asked for."""
    linked = []

    def run(cmd, **kwargs):
        if "-shared" in cmd and cmd[0] == build.HIPCC:
            linked.append(cmd[cmd.index("-o") + 1].split(".tmp.")[0])
            open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setattr(build, "OBJDIR", str(tmp_path / "obj"))
    for name in ("LIB", "BENCH_LIB", "PLAIN_LIB"):
        monkeypatch.setattr(build, name, str(tmp_path / name))
    return linked


def test_the_libraries_need_no_torch(monkeypatch, commands, capsys):
    find = importlib.util.find_spec
    monkeypatch.setattr(importlib.util, "find_spec", lambda name, *a: None if name == "torch" else find(name, *a))

    def no_torch():
        raise ImportError("no torch")
    monkeypatch.setattr(build, "_compile_torch_ext", no_torch)
    assert build.build(verbose=True) == build.LIB
    assert commands == [build.LIB, build.BENCH_LIB, build.PLAIN_LIB]
    assert "torch is not installed" in capsys.readouterr().err


def test_a_torch_binding_that_does_not_compile_fails_after_the_libraries_are_linked(monkeypatch, commands):
    def broken():
        raise RuntimeError("compiling fc_torch.cpp failed")
    monkeypatch.setattr(build, "_compile_torch_ext", broken)
    with pytest.raises(RuntimeError, match="fc_torch.cpp"):
        build.build()
    assert commands == [build.LIB, build.BENCH_LIB, build.PLAIN_LIB]
