"""The build: the C library does not depend on torch or on g++, and an extension of another torch is refused."""
import os
import subprocess
import sys

import pytest

from paper_2406_02540_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def commands(monkeypatch):
    """build.build() with its compilers replaced by a list of what they were asked."""
    seen = []

    class Done:
        def __init__(self, cmd):
            seen.append(cmd)
            self.status = 1 if any(c.endswith("vq_torch.cpp") for c in cmd) and "broken" in cmd else 0

        def wait(self):
            return self.status

    monkeypatch.setattr(build.subprocess, "Popen", Done)
    monkeypatch.setattr(build.subprocess, "check_call", lambda cmd: seen.append(cmd))
    monkeypatch.setattr(build.os, "replace", lambda a, b: seen.append(["replace", a, b]))
    return seen


def test_library_without_torch(commands, monkeypatch):
    monkeypatch.setattr(build.importlib.util, "find_spec", lambda name: None)
    monkeypatch.setitem(sys.modules, "torch", None)   # (an import of it fails)
    assert build.build(verbose=False) == build.LIB_PATH
    assert any(c[0] == "replace" and c[2] == build.LIB_PATH for c in commands)
    assert not any("vq_torch.cpp" in part for c in commands for part in c)


def test_library_is_in_place_before_the_extension(commands, monkeypatch):
    pytest.importorskip("torch")
    monkeypatch.setattr(build, "ext_command", lambda out: ["broken", "vq_torch.cpp"])
    with pytest.raises(RuntimeError, match="vq_torch.cpp"):
        build.build(verbose=False)
    assert [c[2] for c in commands if c[0] == "replace"] == [build.LIB_PATH]


def test_compiler_of_the_extension(monkeypatch, tmp_path):
    monkeypatch.setenv("CXX", "cc1 -m64")
    monkeypatch.setattr(build.shutil, "which", lambda c: "/usr/bin/" + os.path.basename(c) if c in ("cc1", "g++") else None)
    assert build.cxx() == "cc1 -m64"
    monkeypatch.delenv("CXX")
    assert build.cxx() == "g++"
    monkeypatch.setattr(build.shutil, "which", lambda c: c if c.endswith("amdclang++") else None)
    assert build.cxx().endswith("amdclang++")


def test_extension_of_another_torch_is_refused():
    pytest.importorskip("torch")
    if not (os.path.exists(build.LIB_PATH) and os.path.exists(build.EXT_PATH)):
        build.build(verbose=False)
    code = ("import torch; torch.__version__ = '1.0.0+x'; import paper_2406_02540_amd as vq\n"
            "try: vq.vq_quantize_per_token(None)\n"
            "except RuntimeError as e: print('refused', e)\n")
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert out.stdout.startswith("refused") and "build it again" in out.stdout, out.stderr[-2000:]
