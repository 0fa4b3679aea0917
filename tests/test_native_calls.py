"""The extension module between Python and the C ABI, without a GPU: what it hands on and what it refuses."""
import ctypes as C

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
