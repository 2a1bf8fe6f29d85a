"""Which objects a build compiles again: those whose source, headers or command line changed.  The compiler is replaced by one that leaves an
empty object; CPU only."""
import os
import subprocess

import pytest

from paper_2512_18453_amd import build


@pytest.fixture
def compiled(tmp_path, monkeypatch):
    (tmp_path / "csrc").mkdir()
    (tmp_path / "_build").mkdir()
    (tmp_path / "csrc" / "some.hip").write_text("")
    os.utime(tmp_path / "csrc" / "some.hip", (1e9, 1e9))
    monkeypatch.setattr(build, "SRC", str(tmp_path / "csrc"))
    monkeypatch.setattr(build, "OBJ", str(tmp_path / "_build"))
    monkeypatch.setattr(build, "_newest_header", lambda: 1e9)
    calls = []

    def run(cmd, **_):
        calls.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 1 if "-fails" in cmd else 0, "", "")
    monkeypatch.setattr(build.subprocess, "run", run)
    return calls


def test_other_flags_compile_again(compiled, monkeypatch):
    build._compile("some.hip", False)
    build._compile("some.hip", False)
    assert len(compiled) == 1
    for name, value in (("PRELOAD", []), ("COMMON", build.COMMON + ["-DSOME"]), ("DEVICE", build.DEVICE + ["-g"]), ("NO_PRELOAD", ("some.hip",))):
        before = len(compiled)
        monkeypatch.setattr(build, name, value)
        build._compile("some.hip", False)
        build._compile("some.hip", False)
        assert len(compiled) == before + (0 if name == "NO_PRELOAD" else 1), name          # (without PRELOAD the last makes the same command)


def test_objects_of_unknown_or_failed_commands_compile_again(compiled, monkeypatch, tmp_path):
    (tmp_path / "_build" / "some.hip.o").write_text("")                                     # as an older build left it
    build._compile("some.hip", False)
    assert len(compiled) == 1
    monkeypatch.setattr(build, "COMMON", build.COMMON + ["-fails"])
    with pytest.raises(RuntimeError):
        build._compile("some.hip", False)
    monkeypatch.setattr(build, "COMMON", build.COMMON[:-1])
    build._compile("some.hip", False)
    assert len(compiled) == 3
    build._compile("some.hip", True)
    os.utime(tmp_path / "csrc" / "some.hip")
    os.utime(tmp_path / "_build" / "some.hip.o", (1.1e9, 1.1e9))
    build._compile("some.hip", False)
    assert len(compiled) == 5
