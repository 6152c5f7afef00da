"""Deep reductions on the small tiles: with the workspace that the query names (the estimated tile and split), with no more than
select_tile's own choice needs, and at the depth where the estimate begins."""
import ctypes

import pytest
import torch

from paper_2101_08458_amd import unit
from gpu_util import announce

pytestmark = pytest.mark.gpu


class Choice(ctypes.Structure):
    _fields_ = [(f, ctypes.c_int) for f in ("tile", "split_k", "ksteps_per_split", "workgroups")]


def _own_bytes(rows, cols, chunks, dtype, bsrc, cb=0):
    """Bytes of partial sums of select_tile's own choice."""
    fn = unit.load()._ZN4unit11select_tileEiiiiibi
    fn.restype, fn.argtypes = Choice, [ctypes.c_int] * 5 + [ctypes.c_bool, ctypes.c_int]
    split = fn(rows, cols, chunks, dtype, bsrc, True, cb).split_k
    return (split * ((rows * cols + 3) // 4 * 4) * 4 + 255) // 256 * 256 if split > 1 else 0


TYPES = {"i8": torch.int8, "u8i8": torch.uint8, "f16": torch.float16, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}


@pytest.mark.parametrize("dtype", sorted(TYPES))
@pytest.mark.parametrize("m,n,chunks", [(32, 577, 640), (33, 500, 639), (64, 1600, 1001), (150, 700, 1800), (250, 36, 700), (17, 65, 2000)])
def test_products(m, n, chunks, dtype):
    es, ut, ints = (2 if dtype in ("f16", "bf16") else 1), getattr(unit, "UNIT_" + dtype.upper()), dtype in ("i8", "u8i8")
    k = chunks * 16 // es
    g = torch.Generator(device="cuda:0")
    g.manual_seed(m + chunks)
    a = torch.randint(0 if dtype == "u8i8" else -2, 3, (m, k), generator=g, device="cuda:0")
    b = torch.randint(-2, 3, (n, k), generator=g, device="cuda:0")         # (small integers: exact in every type and order)
    exact = a.double() @ b.double().t()
    a, b = a.float().to(TYPES[dtype]), b.float().to(torch.int8 if ints else TYPES[dtype])
    most = unit.unit_matmul_workspace(m, n, k, k, k, ut)
    own = _own_bytes(m, n, chunks, ut, 0) + ((n * 4 + 255) // 256 * 256 if dtype == "u8i8" else 0)
    info = unit.unit_select_matmul(m, n, k, ut)
    assert most >= own and (chunks >= 640 or most == own)
    assert most >= (info.split_k > 1) * info.split_k * m * n * 4
    for size in {most, own, (most + own) // 512 * 256}:
        announce("deep product", dtype, (m, n, k), "workspace", size)
        buf = torch.zeros(size + 256, dtype=torch.uint8, device="cuda:0")
        c = torch.full((m, n), -7, device="cuda:0", dtype=torch.int32 if ints else torch.float32)
        getattr(unit, "unit_matmul_" + dtype)(m, n, k, a, k, b, k, c, n, buf[:size] if size else None)
        torch.cuda.synchronize()
        assert torch.equal(c.double(), exact), size
        assert not buf[size:].any(), "past the workspace"


@pytest.mark.parametrize("dtype", ["i8", "f16"])
@pytest.mark.parametrize("c_bytes,hw,k", [(512, 16, 64), (800, 11, 100), (416, 40, 36)])
def test_convs(c_bytes, hw, k, dtype):
    es, ut = (2 if dtype == "f16" else 1), getattr(unit, "UNIT_" + dtype.upper())
    c = c_bytes // es
    g = torch.Generator(device="cuda:0")
    g.manual_seed(c)
    x = torch.randint(-2, 3, (2, c, hw, hw), generator=g, device="cuda:0")
    w = torch.randint(-2, 3, (k, c, 5, 5), generator=g, device="cuda:0")
    exact = torch.nn.functional.conv2d(x.double(), w.double(), padding=2, stride=2)
    d = unit.conv_desc(2, c, hw, hw, k, 5, 5, 2, 2)
    x, w = x.float().to(TYPES[dtype]), w.float().to(TYPES[dtype])
    wp = torch.empty(unit.unit_packed_weights_bytes(d, ut), dtype=torch.uint8, device="cuda:0")
    getattr(unit, "unit_pack_weights_" + dtype)(d, w, wp)
    most = unit.unit_conv2d_wpacked_workspace(d, ut)
    own = unit.unit_packed_act_bytes(2, c, hw, hw, ut) + _own_bytes(k, exact.numel() // k, 25 * c_bytes // 16, ut, 1, c_bytes // 16)
    for size in {most, own}:
        announce("deep conv", dtype, (c, hw, k), "workspace", size)
        buf = torch.zeros(size + 256, dtype=torch.uint8, device="cuda:0")
        y = torch.full(exact.shape, -7, device="cuda:0", dtype=torch.int32 if dtype == "i8" else torch.float32)
        if dtype == "i8":
            unit.unit_conv2d_wpacked_i8(d, x, wp, y, None, None, buf[:size])
        else:
            unit.unit_conv2d_wpacked_f16(d, x, wp, y, buf[:size])
        torch.cuda.synchronize()
        assert torch.equal(y.double(), exact), size
        assert not buf[size:].any(), "past the workspace"
