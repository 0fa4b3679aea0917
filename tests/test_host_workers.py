"""The worker threads of the host functions: calls from several threads, a forked child, and a library that is unloaded
or a process that ends while they are still there.  Each in a child process of its own (a fault there ends the child,
not the test run)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2605_11582_amd", "libegt.so")

COMMON = r"""
import ctypes as C, os, sys, threading, time, _ctypes
import numpy as np
L = C.CDLL({lib!r})                                       # (without PyTorch: nothing else keeps the library loaded)
L.egt_prune_n4.argtypes = [C.c_void_p, C.c_int64, C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_int64]
rows, cols = 2048, 2048                                   # enough work for every worker
def weights(seed):
    return np.random.default_rng(seed).standard_normal((rows, cols)).astype(np.float16).view(np.uint16)
def prune(w):
    mask = np.empty((rows, cols), dtype=np.uint8)
    assert L.egt_prune_n4(w.ctypes.data, cols, rows, cols, 2, mask.ctypes.data, cols) == 0
    return mask
def want(w):
    m = (w & 0x7FFF).reshape(rows, -1, 4).astype(np.int32)
    order = np.argsort(-m, axis=-1, kind="stable")[..., :2]
    out = np.zeros_like(m, dtype=np.uint8)
    np.put_along_axis(out, order, 1, axis=-1)
    return out.reshape(rows, cols)
def threads():
    return len(os.listdir("/proc/self/task"))
"""

UNLOAD = r"""
prune(weights(0))
_ctypes.dlclose(L._handle)
mapped = open("/proc/self/maps").read().count("libegt.so")
time.sleep(0.5)                                           # (idle workers look around after a fifth of a second)
print("mapped", mapped)
"""

UNLOAD_AND_LOAD = r"""
w = weights(0)
ref = want(w)
for k in range(5):
    assert np.array_equal(prune(w), ref)
    time.sleep((0, 0.19, 0.2, 0.21, 0)[k])                # (workers that are just leaving, too)
    _ctypes.dlclose(L._handle)
    L = C.CDLL({lib!r})
    L.egt_prune_n4.argtypes = [C.c_void_p, C.c_int64, C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_int64]
assert np.array_equal(prune(w), ref)
"""

LEAVE = r"""
w = weights(0)
before = threads()
prune(w)
time.sleep(0.6)
assert threads() == before, (threads(), before)
assert np.array_equal(prune(w), want(w))                  # and are started again
time.sleep(0.6)
assert threads() == before, (threads(), before)
"""

TWO = r"""
ws = [weights(k) for k in range(3)]
refs = [want(w) for w in ws]
bad = []
def body(k):
    for _ in range(12):
        if not np.array_equal(prune(ws[k]), refs[k]):
            bad.append(k)
ts = [threading.Thread(target=body, args=(k,)) for k in range(3)]
for t in ts: t.start()
for t in ts: t.join()
assert not bad
assert threads() <= 16 + 4, threads()
"""

FORK = r"""
w = weights(0)
ref = want(w)
prune(w)                                                  # (the workers are there when the process forks)
pid = os.fork()
ok = all(np.array_equal(prune(w), ref) for _ in range(3))
if pid == 0:
    sys.exit(0 if ok else 3)                              # (by the way that runs the library's own end)
assert ok
assert os.waitpid(pid, 0)[1] == 0
"""

LAST = r"""
w = weights(0)
prune(w)                                                  # the process ends with the workers waiting
"""

DAEMON = r"""
w = weights(0)
prune(w)
def body():
    while True: prune(w)
threading.Thread(target=body, daemon=True).start()
time.sleep(0.1)                                           # the process ends with a call on its way
"""


@pytest.mark.parametrize("what", ["UNLOAD", "UNLOAD_AND_LOAD", "LEAVE", "TWO", "FORK", "LAST", "DAEMON"])
def test_worker_threads(what):
    code = (COMMON + globals()[what]).replace("{lib!r}", repr(LIB))
    run = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, (run.returncode, run.stdout[-1500:], run.stderr[-1500:])
    if what == "UNLOAD":
        assert run.stdout.split() == ["mapped", "0"], run.stdout
