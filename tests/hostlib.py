"""Compiles host code that includes the kernels' headers, for tests of the rules that host and device share."""
import ctypes
import subprocess

from paper_2503_04558_amd import build


def host_library(tmp_path, name: str, source: str) -> ctypes.CDLL:
    src, out = tmp_path / f"{name}.hip", tmp_path / f"{name}.so"
    src.write_text(source)
    subprocess.check_call([build.HIPCC, "-O2", "-std=c++17", "--offload-host-only", "-fPIC", "-shared", "-I",
                           build.INCLUDE, "-I", build.CSRC, str(src), "-o", str(out)])
    return ctypes.CDLL(str(out))
