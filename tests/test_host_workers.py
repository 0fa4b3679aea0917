"""The worker threads of the host functions: calls from several threads, a forked child, and a library that is unloaded
or a process that ends while they are still there.  Each in a child process of its own (a fault there ends the child,
not the test run)."""
import os
import shutil
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

FORK_AFTER_UNLOAD = r"""
prune(weights(0))
_ctypes.dlclose(L._handle)
pid = os.fork()                                           # (nothing of the library is called in the child any more)
if pid == 0:
    os._exit(0)
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


@pytest.mark.parametrize("what", ["UNLOAD", "UNLOAD_AND_LOAD", "LEAVE", "TWO", "FORK", "FORK_AFTER_UNLOAD", "LAST", "DAEMON"])
def test_worker_threads(what):
    code = (COMMON + globals()[what]).replace("{lib!r}", repr(LIB))
    run = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, (run.returncode, run.stdout[-1500:], run.stderr[-1500:])
    if what == "UNLOAD":
        assert run.stdout.split() == ["mapped", "0"], run.stdout


NO_MEMORY = r"""
#include "egt.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>
static bool armed = false;
void *operator new(size_t n) { void *p = armed ? nullptr : std::malloc(n); if (!p) throw std::bad_alloc(); return p; }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
int main() {
  const int R = 1024, K = 1024;
  for (int kind = 0; kind < 3; ++kind) for (int group : {128, 12, 4}) {
    const int cols = group == 12 ? 960 : K, gr = kind == EGT_VAL_FP16 ? 0 : group;
    std::vector<uint16_t> w(R * K);
    for (size_t i = 0; i < w.size(); ++i) w[i] = (uint16_t)((i * 2654435761u >> 13) & 0xBBFF);
    struct Out { std::vector<uint8_t> mask, v, q, m2; std::vector<uint16_t> ix, qp, d, dqp; std::vector<uint32_t> rp; };
    Out o[2];
    for (Out &x : o) { x.mask.resize(R * K); x.v.resize(R * K); x.q.resize(R * K); x.m2.resize(R * K); x.ix.resize(R * K); x.qp.resize(R * K); x.d.resize(R * K); x.dqp.resize(R * K); x.rp.resize(R + 1); }
    for (int k = 0; k < 2; ++k) {
      Out &x = o[k];
      egt_2bitcsr p{};
      p.row_ptr = x.rp.data(); p.values = x.v.data(); p.idx = x.ix.data(); p.qparams = x.qp.data();
      armed = k == 1;                                    // no memory, and no thread, to be had
      int st = egt_prune_n4(w.data(), K, R, cols, 2, x.mask.data(), K);
      st |= egt_pack_2bitcsr(w.data(), K, x.mask.data(), K, R, cols, 2, gr, kind, &p);
      st |= egt_unpack_2bitcsr(&p, x.d.data(), K, x.m2.data(), K);
      if (kind != EGT_VAL_FP16) st |= egt_quant_int4(w.data(), K, R, cols, group, x.q.data(), x.dqp.data());
      armed = false;
      if (st) { std::printf("status %d\n", st); return 1; }
    }
    if (o[0].mask != o[1].mask || o[0].v != o[1].v || o[0].q != o[1].q || o[0].m2 != o[1].m2 || o[0].ix != o[1].ix || o[0].qp != o[1].qp ||
        o[0].d != o[1].d || o[0].dqp != o[1].dqp || o[0].rp != o[1].rp) { std::puts("other bytes"); return 1; }
  }
  std::puts("ok");
}
"""


@pytest.mark.parametrize("first", [False, True])
def test_host_functions_without_memory(first, tmp_path):
    """No C++ exception leaves a host function, and none ends a worker: the parts of a job allocate nothing."""
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "nomem.cpp", str(tmp_path / "nomem")
    # `first`: not even the first call has memory, so no worker is ever started
    src.write_text(NO_MEMORY.replace("k == 1", "true") if first else NO_MEMORY)
    build = subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-ffp-contract=off", "-I" + os.path.join(ROOT, "include"), str(src),
                            os.path.join(ROOT, "paper_2605_11582_amd", "csrc", "egt_host.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.split() == ["ok"], (run.returncode, run.stdout[-500:], run.stderr[-500:])
