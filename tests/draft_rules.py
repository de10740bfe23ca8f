"""The size rules of the draft calls, compiled from csrc/draft_rules.h with the host compiler: what the library decides on a
device of any number of compute units, without one."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(maxsize=None)
def rules():
    tmp = tempfile.mkdtemp()
    lib = os.path.join(tmp, "draft_rules.so")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2511_14102_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "draft_rules.cpp"), "-o", lib], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(lib)
