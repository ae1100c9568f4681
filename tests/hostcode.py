"""Host headers of the library compiled on their own (g++), for tests of the rules that they
hold."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_11673_amd", "csrc")


def compiled(tmp_path, source):
    src, lib = tmp_path / "t.cpp", tmp_path / "t.so"
    src.write_text(source)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src),
                           "-o", str(lib)])
    return ctypes.CDLL(str(lib))
