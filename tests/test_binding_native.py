"""The binding's native argument conversions against the ctypes ones: the same status, refusals and exceptions (no GPU: every call
is refused on the host before its first HIP call, or compares the conversion alone)."""
import ctypes
import os

import pytest

from paper_2101_08458_amd import unit


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(unit.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    unit.load()


class Tensor:
    def __init__(self, ptr, n=1 << 20):
        self.ptr, self.n = ptr, n

    def data_ptr(self):
        return self.ptr

    def numel(self):
        return self.n

    def element_size(self):
        return 2


class Stream:
    cuda_stream = 0


RET = ctypes.c_int


def _seen(kind, nargs, values):
    """Arguments a C function of nargs words gets from a native entry."""
    from paper_2101_08458_amd import _unitcall
    got = []
    types = {"matmul": [ctypes.c_int32] * 3 + [ctypes.c_void_p, ctypes.c_int64] * 3 + [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p],
             "conv": [ctypes.c_void_p] * 5 + [ctypes.c_size_t, ctypes.c_void_p],
             "conv_i8": [ctypes.c_void_p] * 7 + [ctypes.c_size_t, ctypes.c_void_p],
             "packed_i8": [ctypes.c_void_p] * 8 + [ctypes.c_size_t, ctypes.c_void_p]}[kind]
    fn = ctypes.CFUNCTYPE(RET, *types)(lambda *a: got.append(a) or -3)
    entry = _unitcall.entry(kind, ctypes.cast(fn, ctypes.c_void_p).value, unit.unit_conv2d_desc, unit.unit_requant)
    return entry(*values), got[0] if got else None


def test_arguments_arrive():
    A, ws, d, rq = Tensor((1 << 47) + 16), Tensor(4096, 100), unit.conv_desc(1, 2, 3, 4, 5, 1, 1), unit.make_requant(16)
    p = ctypes.addressof
    assert _seen("matmul", 12, (-1, 2 ** 31 - 1, True, A, 1 << 40, 64, -5, None, 7, ws, 9)) == (
        -3, (-1, 2 ** 31 - 1, 1, A.ptr, 1 << 40, 64, -5, None, 7, 4096, 200, 9))
    assert _seen("conv", 7, (d, A, None, ws, None, Stream())) == (-3, (p(d), A.ptr, None, 4096, None, 0, None))
    assert _seen("conv_i8", 9, (d, A, A, None, rq, ws, ws, 8)) == (-3, (p(d), A.ptr, A.ptr, None, p(rq), 4096, 4096, 200, 8))
    assert _seen("packed_i8", 10, (d, A, A, A, None, None, ws, None, 8)) == (-3, (p(d), A.ptr, A.ptr, A.ptr, None, None, 4096, None, 0, 8))


def test_anything_else_is_left_to_ctypes():
    A, d = Tensor(64), unit.conv_desc(1, 2, 3, 4, 5, 1, 1)
    good = [1, 2, 3, A, 4, A, 5, A, 6, None, 7]
    for at, v in [(0, 2 ** 31), (1, 1.0), (2, "3"), (4, 1 << 63), (3, -1), (10, -1)]:
        a = list(good)
        a[at] = v
        assert _seen("matmul", 12, a) == (None, None), (at, v)
    d3 = unit.conv3d_desc(1, 2, 3, 4, 5, 1, 1, 1, 1)
    assert _seen("conv", 7, (d3, A, A, A, None, 0)) == (None, None)
    assert _seen("conv_i8", 9, (d, A, A, A, d, A, None, 0)) == (None, None)
    with pytest.raises(AttributeError):
        _seen("conv", 7, (d, object(), A, A, None, 0))
    with pytest.raises(TypeError):
        _seen("conv", 7, (d, A, A))


def test_public_calls_refuse_as_before():
    A, d = Tensor(256), unit.conv_desc(1, 2, 3, 4, 5, 9, 9)
    for call in (lambda: unit.unit_matmul_i8(0, 2, 3, A, 3, A, 3, A, 2, None, 0), lambda: unit.unit_conv2d_f16(d, A, A, A, None, 0),
                 lambda: unit.unit_conv2d_i8(d, A, A, A, None, None, None, 0), lambda: unit.unit_conv2d_packed_i8(d, A, A, A, None, None, None, None, 0)):
        with pytest.raises(unit.UnitError) as e:
            call()
        assert e.value.status == unit.UNIT_EINVAL
    with pytest.raises(ctypes.ArgumentError):
        unit.unit_matmul_i8(1.5, 2, 3, A, 3, A, 3, A, 2, None, 0)
