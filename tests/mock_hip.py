"""Runs a piece of Python against the library with mock_hip.c in front of the HIP
runtime (a process of its own), and returns what it printed. The piece finds
``lib`` (the library), ``mock`` (the stand-in) and ``kernels()`` (the short names of
the kernels launched since the last mock_reset)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = """
import ctypes, re, sys
sys.path.insert(0, %r)
mock = ctypes.CDLL(%r)
mock.mock_reset.argtypes = [ctypes.c_size_t]
mock.mock_log.restype = ctypes.c_char_p
mock.mock_largest.restype = ctypes.c_size_t
import numpy as np
from paper_1905_13298_amd import _native
lib = _native.lib()
ALL = (1 << 64) - 1
def kernels():
    return [re.match(r"_ZN2ds(?:12_GLOBAL__N_1)?\\d+([a-z_0-9]*kernel)", n).group(1) if "kernel" in n else n
            for n in mock.mock_log().decode().split()]
"""


def run(piece: str, tmp_path) -> str:
    so = str(tmp_path / "mock_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", "-o", so, os.path.join(ROOT, "tests", "mock_hip.c")],
                   check=True)
    env = dict(os.environ, LD_PRELOAD=so)
    res = subprocess.run([sys.executable, "-c", HEAD % (ROOT, so) + piece], cwd=ROOT, env=env, capture_output=True,
                         text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    return res.stdout
