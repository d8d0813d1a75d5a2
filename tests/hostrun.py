"""Runs a snippet against the library's host code on the CPU: a child process loads fake_hip.c as the
HIP runtime, then the library, and the snippet prints what it found as JSON.

Names in the snippet: np, I (inputs), lbm, fake (the runtime's own questions), launches() (the
list of (kernel, workgroups, first, second pointer argument) launched since it was last asked), case(...)
(a box at rest) and result(value), which ends it."""
import ctypes
import functools
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
_DIR = tempfile.TemporaryDirectory(prefix="lbm_fake_hip_")

_PRELUDE = r'''
import ctypes, json, re, sys
sys.path[:0] = [{root!r}, {here!r}]
fake = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
fake.fake_held.restype = fake.fake_peak.restype = ctypes.c_size_t
fake.fake_capacity.argtypes = [ctypes.c_size_t]
import numpy as np
from paper_1705_10045_amd import inputs as I
from paper_1705_10045_amd import lbm

def launches():
    out = []
    for line in fake.fake_log().decode().splitlines():
        name, blocks, a, b = line.rsplit(" ", 3)
        m = re.search(r"k_[a-z_]*[a-z]", name)
        out.append((m.group(0) if m else name, int(blocks), a, b))
    return out

def case(Q, shape, storage=4, **kw):
    args = (Q, I.physics(**kw), np.full(shape, 0.2), np.zeros((3,) + tuple(shape)), np.full(shape, 0.85))
    return lbm.Sim(*args, storage_bytes=storage)

def result(value):
    print("RESULT " + json.dumps(value))
'''


@functools.lru_cache(maxsize=1)
def _runtime():
    out = os.path.join(_DIR.name, "libamdhip64.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", "-Wl,-soname,libamdhip64.so.7",
                    "-Wl,--version-script," + os.path.join(HERE, "fake_hip.map"), "-o", out,
                    os.path.join(HERE, "fake_hip.c"), "-lpthread"], check=True)
    return out


def run(snippet):
    code = _PRELUDE.format(root=ROOT, here=HERE, lib=_runtime()) + snippet
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    lines = [line for line in r.stdout.splitlines() if line.startswith("RESULT ")]
    assert r.returncode == 0 and lines, r.stdout + r.stderr
    return json.loads(lines[-1][len("RESULT "):])
