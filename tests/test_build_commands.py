"""The commands that paper_2603_08088_amd.build would run (nothing is compiled here)."""
import os

import pytest

from paper_2603_08088_amd import build


@pytest.fixture
def commands(monkeypatch, tmp_path):
    seen = []
    monkeypatch.setattr(build, "_run", lambda cmd, verbose: seen.append(cmd))
    monkeypatch.setattr(build, "BINDING", str(tmp_path / "_binding.so"))
    return seen


@pytest.mark.parametrize("hipcc", ["hipcc", "/opt/rocm/bin/hipcc"])
def test_hip_headers_are_found_by_the_compilers_path_and_by_its_name(commands, monkeypatch, hipcc):
    monkeypatch.setattr(build, "HIPCC", hipcc)
    monkeypatch.setenv("PATH", "/opt/rocm/bin" + os.pathsep + os.environ["PATH"])
    build.build()
    assert len(commands) == 3 and commands[2][-1].startswith("-Wl,-rpath")
    includes = [a[2:] for a in commands[2] if a.startswith("-I")]
    assert any(os.path.exists(os.path.join(d, "hip", "hip_runtime_api.h")) for d in includes), includes


def test_library_is_built_without_a_host_compiler(commands, monkeypatch, capsys):
    monkeypatch.setenv("CXX", "no-such-compiler")
    open(build.BINDING, "w").close()
    assert build.build() == build.LIB
    assert [c[-1] for c in commands] == [build.LIB, build.PROBE_LIB]      # both libraries, nothing else
    assert "no-such-compiler" in capsys.readouterr().out and not os.path.exists(build.BINDING)


def test_library_is_built_without_torch(commands, monkeypatch, capsys):
    monkeypatch.setattr(build.importlib.util, "find_spec", lambda name: None)
    build.build()
    assert [c[-1] for c in commands] == [build.LIB, build.PROBE_LIB] and "torch" in capsys.readouterr().out
