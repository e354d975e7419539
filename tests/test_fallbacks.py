"""What the package takes from torch's and the compiler's insides is not needed:
without it the public way is taken."""
import os
import subprocess
import types

import pytest
import torch

from paper_2503_04558_amd import build, grpic


def test_stream_without_the_raw_getter(monkeypatch):
    monkeypatch.setattr(grpic, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=123))
    assert grpic._stream(None) == 123
    assert grpic._stream(7) == 7 and grpic._stream(types.SimpleNamespace(cuda_stream=9)) == 9


def test_stream_takes_the_current_device(monkeypatch):
    monkeypatch.setattr(grpic, "_raw_stream", lambda device: 1000 + device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert grpic._stream(None) == 1003


def _compiler(path, body):
    path.write_text("#!/bin/sh\n" + body)
    os.chmod(path, 0o755)
    return str(path)


def test_build_without_the_compilers_switches(tmp_path, monkeypatch):
    """A compiler that refuses -mllvm switches still builds every source; one that refuses everything raises."""
    log = tmp_path / "log"
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "HIPCC", _compiler(tmp_path / "cc", f'echo "$@" >> {log}\ncase "$*" in *-mllvm*) exit 1;; esac\n'))
    src = os.path.join(build.CSRC, "adjoint.hip")
    assert build._compile(src, False) == str(tmp_path / "adjoint.hip.o")
    tried = log.read_text().splitlines()
    assert len(tried) == 2 and "-mllvm" in tried[0] and "-mllvm" not in tried[1]
    assert "-packed-fp32-ops" in tried[1] and "--offload-arch=gfx950" in tried[1]
    build._compile(os.path.join(build.CSRC, "sort.hip"), False)
    assert len(log.read_text().splitlines()) == 3
    monkeypatch.setattr(build, "HIPCC", _compiler(tmp_path / "bad", "exit 3\n"))
    with pytest.raises(subprocess.CalledProcessError):
        build._compile(src, False)
