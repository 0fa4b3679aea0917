"""The extension module between Python and the C ABI, without a GPU: what it hands on and what it refuses."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2605_11582_amd import binding as egt

READ = C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_size_t, C.c_void_p, C.c_void_p)


@pytest.mark.parametrize("given,seen", [((), 7), ((9,), 9), ((None,), None), ((C.c_void_p(11),), 11), ((C.c_void_p(),), None)])
def test_stream_argument_of_a_prepared_call(given, seen):
    got = []

    def entry(src, nbytes, sink, stream):
        got.append((src, nbytes, sink, stream))
        return 0
    fn = READ(entry)
    call = egt._native().Call(egt._native().READ, C.cast(fn, C.c_void_p).value, [(1, 2, 3)], 7, None)
    call(*given)
    assert got == [(1, 2, 3, seen)]
    if given:
        call(stream_ptr=given[0])
        assert got[1] == got[0]


def test_stream_argument_of_the_wrong_type():
    fn = READ(lambda *a: pytest.fail("launched"))
    call = egt._native().Call(egt._native().READ, C.cast(fn, C.c_void_p).value, [(1, 2, 3)], 7, None)
    for bad in ("0", 1.5, object()):
        with pytest.raises(TypeError):
            call(bad)


def test_prepared_calls_are_referred_to_and_copied_like_functions():
    import copy
    import gc
    import weakref

    class Kept:
        pass
    kept = Kept()
    fn = READ(lambda *a: 0)
    call = egt._native().Call(egt._native().READ, C.cast(fn, C.c_void_p).value, [(1, 2, 3)], 7, [kept])
    call.plan = {"count": 1}
    assert copy.copy(call) is call and copy.deepcopy({"step": [call]})["step"][0] is call
    ref, kept_ref = weakref.ref(call), weakref.ref(kept)
    table = weakref.WeakKeyDictionary({call: 1})
    assert ref() is call and table[call] == 1
    call.itself = call                                    # (a cycle)
    del call, kept
    gc.collect()
    assert ref() is None and kept_ref() is None and not table


NO_MEMORY = r"""
#include <cstdlib>
#include <new>
static bool armed = false;
extern "C" void arm(int on) { armed = on != 0; }
void *operator new(size_t n) { void *p = armed ? nullptr : std::malloc(n ? n : 1); if (!p) throw std::bad_alloc(); return p; }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
"""
CHILD = r"""
import ctypes, sys
sys.path.insert(0, {root!r})
from paper_2605_11582_amd import binding as egt
native, arm = egt._native(), ctypes.CDLL({lib!r}).arm
args = (native.READ, 1 << 20, [(1, 2, 3)], 7, None)
native.Call(*args)
arm(1)
try:
    native.Call(*args)
    print("made")
except MemoryError:
    print("no memory")
arm(0)
native.Call(*args)
"""


def test_a_prepared_call_without_memory_is_a_memory_error(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")
    lib, root = str(tmp_path / "nomem.so"), os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    (tmp_path / "nomem.cpp").write_text(NO_MEMORY)
    subprocess.run([gxx, "-shared", "-fPIC", "-O1", str(tmp_path / "nomem.cpp"), "-o", lib], check=True)
    env = dict(os.environ)
    env["LD_PRELOAD"] = " ".join(v for v in (lib, env.get("LD_PRELOAD", "")) if v)
    run = subprocess.run([sys.executable, "-c", CHILD.replace("{root!r}", repr(root)).replace("{lib!r}", repr(lib))],
                         capture_output=True, text=True, env=env, timeout=120)
    assert run.returncode == 0 and run.stdout.split("\n")[0] == "no memory", (run.returncode, run.stdout[-300:], run.stderr[-800:])


def test_tensors_without_memory_are_left_to_the_checks():
    """The elements of a batch under vmap have no memory of their own: asking for their address throws in C++."""
    from torch._subclasses.fake_tensor import FakeTensorMode
    native = egt._native()

    def body(t, t2):
        p = egt.Packed(64, 64, 2, 64, egt.VAL_INT4, t, t, t, t)
        assert native.sparse_gemv(p, t, t, None) is False
        assert native.sparse_gemm_smallm(0, p, t2, t2, None, None) is False
        assert native.int4_gemv(t, t, 64, 64, 64, t, t, None) is False
        return t
    with FakeTensorMode():                                # (device tensors without a device)
        torch.vmap(body)(torch.empty((3, 4096), dtype=torch.float16, device="cuda"),
                         torch.empty((3, 4, 64), dtype=torch.float16, device="cuda"))


@pytest.mark.gpu
def test_an_error_of_the_hip_runtime_is_raised_by_the_call_that_meets_it():
    """Entry points that fail once with a HIP error: one call, one exception; nothing is tried again in silence."""
    calls = []
    types = {"egt_sparse_gemv": C.CFUNCTYPE(C.c_int, *[C.c_void_p] * 4),
             "egt_sparse_gemm_smallm": C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_int64, C.c_int, C.c_void_p),
             "egt_sparse_gemm_smallm_ws": C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_int64, C.c_int, C.c_void_p, C.c_size_t, C.c_void_p),
             "egt_int4_gemv": C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_void_p)}
    types["egt_sparse_gemm_smallm_static"] = types["egt_sparse_gemm_smallm"]

    def failing(name):
        def entry(*a):
            calls.append(name)
            return 7
        return types[name](entry)
    fns = [failing(name) for name in egt._plain]
    native = egt._native()
    t = torch.zeros(1 << 16, dtype=torch.float16, device="cuda")
    p = egt.Packed(64, 64, 2, 64, egt.VAL_INT4, t, t, t, t)
    X, Y = t[:256].view(4, 64), t[:256].view(4, 64)
    native.bind(*[C.cast(f, C.c_void_p).value for f in fns], egt._check, torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice)
    try:
        for call in (lambda: egt.sparse_gemv(p, t, t), lambda: egt.int4_gemv(t, t, 64, 64, 64, t, t), lambda: egt.sparse_gemm_smallm(p, X, Y),
                     lambda: egt.sparse_gemm_smallm_ws(p, X, Y, None), lambda: egt.sparse_gemm_smallm_static(p, X, Y)):
            with pytest.raises(egt.EgtError) as e:
                call()
            assert e.value.status == 7 and len(calls) == 1, calls
            calls.clear()
    finally:
        egt._call = None
        egt._native()
