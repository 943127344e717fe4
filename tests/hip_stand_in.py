"""Runs libge's host side in a child process over fake_hip.c, so that tests on the
CPU see what it would enqueue."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# what every child starts with: the stand-in, then the library.  log(): one
# [what, stream, event, thread, workgroups, threads] per call
HEAD = """
import ctypes, json, sys, threading
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
from paper_1310_3422_amd import ge
def table(sizes):
    n = np.array(sizes, dtype=np.int64)
    off = np.zeros(n.size + 1, dtype=np.int64)
    off[1:] = np.cumsum((n + 3) // 4 * 4)
    one = np.ones(n.size)
    return n, off, one, 0 * one, 0 * one
def log():
    return [l.split() for l in fake.fake_log().decode().splitlines()]
"""


def child(tmp_path, code):
    """The JSON value that `code` prints last."""
    so = os.path.join(str(tmp_path), "fake_hip.so")
    if not os.path.exists(so):
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so,
                        os.path.join(ROOT, "tests", "fake_hip.c"), "-lpthread"], check=True)
    r = subprocess.run([sys.executable, "-c", HEAD + code, so], cwd=ROOT, capture_output=True,
                       text=True, timeout=120, env={**os.environ, "GE_TUNE_CACHE": "/nonexistent"})
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    return json.loads(r.stdout.splitlines()[-1])
