"""The library's host side on the runtime in host memory (fake_hip.cpp):
``run(script)`` runs a script in a process of its own, in which ``m`` is the
binding and ``fake`` the runtime's own controls."""
import functools
import os
import subprocess
import sys
import tempfile

from paper_2102_05297_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

_PROLOGUE = """
import ctypes
fake = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
fake.fake_used.restype = ctypes.c_size_t
fake.fake_limit.argtypes = fake.fake_host_limit.argtypes = [ctypes.c_size_t]
import numpy as np
from paper_2102_05297_amd import cgs as m

def log():
    return [l.split() for l in fake.fake_log().decode().splitlines()]

def space(*radix):
    return m.Space(list(radix), [list(range(1, r + 1)) for r in radix])

def forest(sp, C, value=1.0):
    return m.ForestModel(sp, np.zeros((1, 0), np.uint8), np.zeros((1, 0), np.uint8),
                         np.full((1, 1, C), value, np.float32))

def status(call):
    try:
        call()
        return 0
    except m.CgsError as e:
        return e.status

U = np.arange(1, 4000, dtype=np.uint64)
"""


@functools.lru_cache(None)
def library() -> str:
    out = os.path.join(tempfile.mkdtemp(prefix="fake_hip"), "libfake_hip.so")
    rocm = os.path.dirname(os.path.dirname(build.hipcc()))
    subprocess.run([os.path.join(rocm, "bin", "amdclang++"), "-D__HIP_PLATFORM_AMD__", "-std=c++17", "-O1", "-fPIC",
                    "-shared", f"-I{rocm}/include", f"-I{build.INCLUDE}", f"-I{build.CSRC}",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", out], check=True)
    return out


def run(script: str) -> None:
    code = _PROLOGUE.format(lib=library()) + script
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
