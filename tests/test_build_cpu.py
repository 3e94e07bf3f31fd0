"""build_lib.build() with its compilers replaced by stand-ins that only record
their commands: the C library needs hipcc alone."""

import subprocess
import sys

import pytest

from paper_2108_02347_amd import build_lib


class _Process:
    returncode = 0
    stdout = stderr = ""

    def __init__(self, cmd, **_):
        self.args = cmd
        open(cmd[cmd.index("-o") + 1], "w").close()

    def communicate(self):
        return "", None


@pytest.mark.parametrize("torch_there", [True, False])
def test_library_builds_without_torch(monkeypatch, tmp_path, torch_there):
    cmds = []

    def start(cmd, **kw):
        cmds.append(cmd)
        return _Process(cmd, **kw)

    monkeypatch.setattr(build_lib, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build_lib, "TORCH_EXT", str(tmp_path / "ext.so"))
    monkeypatch.setattr(subprocess, "Popen", start)
    monkeypatch.setattr(subprocess, "run", start)
    if not torch_there:
        monkeypatch.setitem(sys.modules, "torch", None)  # the import raises ImportError
    assert build_lib.build() == str(tmp_path / "lib.so")
    assert (tmp_path / "lib.so").exists()
    assert (tmp_path / "ext.so").exists() == torch_there
    assert any("fmm_torch.cpp" in x for cmd in cmds for x in cmd) == torch_there
    assert sum(any(x.endswith(".hip") for x in cmd) for cmd in cmds) >= len(build_lib.SOURCES) - 1


def test_library_stays_when_the_extension_fails(monkeypatch, tmp_path):
    def start(cmd, **kw):
        p = _Process(cmd, **kw)
        p.returncode = int(any("fmm_torch.cpp" in x for x in cmd))
        return p

    monkeypatch.setattr(build_lib, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build_lib, "TORCH_EXT", str(tmp_path / "ext.so"))
    monkeypatch.setattr(subprocess, "Popen", start)
    monkeypatch.setattr(subprocess, "run", start)
    with pytest.raises(RuntimeError):
        build_lib.build()
    assert (tmp_path / "lib.so").exists()
