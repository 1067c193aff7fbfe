"""Runs code against the library in a process without a GPU, on the host
memory runtime of host_hip.c: launches are recorded, not run."""
from __future__ import annotations

import functools
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

_HEAD = """
import ctypes, json, sys
H = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
H.host_hip_log.restype = ctypes.c_char_p
H.host_hip_used.restype = ctypes.c_longlong
H.host_hip_limit.argtypes = [ctypes.c_longlong]
H.host_hip_slow.argtypes = [ctypes.c_char_p]
sys.path.insert(0, sys.argv[2])
import paper_1908_06091_amd as P
L = P.lib()
IN, OUT, OUT2 = 1 << 42, 1 << 43, 1 << 44  # field addresses: never read
F64, F32 = P.ATLAS_F64, P.ATLAS_F32
GRAD, DIV, CURL, LAPL = 0, 1, 2, 3

def launches(fn, *args):
    # [name, blocks, threads, LDS bytes] of every kernel the call launches
    H.host_hip_clear()
    rc = fn(*args)
    assert rc == 0, (rc, L.atlas_last_error())
    return [[f if i == 0 else int(f) for i, f in enumerate(l.split())]
            for l in H.host_hip_log().decode().splitlines()]

def apply(m, op, nlev, dtype, launch=None):
    return launches(L.atlas_nabla_apply, m.handle, op, IN, nlev, dtype, OUT, None,
                    None if launch is None else ctypes.byref(launch), None)

"""


@functools.lru_cache(maxsize=None)
def _runtime():
    so = os.path.join(tempfile.mkdtemp(prefix="host_hip"), "libhost_hip.so")
    subprocess.run(["gcc", "-O1", "-std=c11", "-D_DEFAULT_SOURCE", "-fPIC", "-shared", "-o", so,
                    os.path.join(HERE, "host_hip.c")], check=True)
    return so


def on_host(code: str):
    """`result` of the Python `code`, run in a process of its own."""
    p = subprocess.run([sys.executable, "-c", _HEAD + code + "\nprint(json.dumps(result))",
                        _runtime(), ROOT], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr[-3000:]
    return json.loads(p.stdout.splitlines()[-1])
