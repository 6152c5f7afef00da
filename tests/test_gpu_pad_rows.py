"""Operand rows the matmul cannot read in place (odd widths, pitches and addresses): copied, zero filled and multiplied.  One
operand or both, rows of less than one 16-byte chunk to several, what lies between the rows and beside the matrix poisoned."""
import pytest
import torch

from paper_2101_08458_amd import unit
from gpu_util import announce

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def matrix(g, dtype, rows, k, ld, offset):
    """[rows][k] at an offset (in elements) inside a buffer whose other elements would spoil every sum they entered."""
    if dtype == torch.int8:
        buf = torch.full((rows * ld + offset,), 127, dtype=dtype, device=DEV)
        vals = torch.randint(-128, 128, (rows, k), generator=g, device=DEV, dtype=dtype)
    else:
        buf = torch.full((rows * ld + offset,), float("nan"), dtype=dtype, device=DEV)
        vals = torch.randint(-8, 9, (rows, k), generator=g, device=DEV).to(dtype)        # sums are exact in fp32
    view = buf[offset:].view(rows, ld)
    view[:, :k] = vals
    return view, vals


@pytest.mark.parametrize("dtype", [torch.int8, torch.float16])
@pytest.mark.parametrize("m,n,k,lda,ldb,offset", [
    (1, 65, 7, 7, 7, 1), (33, 70, 15, 19, 16, 0), (40, 1, 17, 17, 21, 3), (130, 50, 129, 129, 160, 0), (50, 130, 144, 144, 145, 0),
    (257, 300, 1777, 1777, 1781, 5), (3, 900, 31, 48, 31, 0), (64, 64, 16, 17, 33, 9)])
def test_unaligned_rows(dtype, m, n, k, lda, ldb, offset):
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    ut, fn, out = ((unit.UNIT_I8, unit.unit_matmul_i8, torch.int32) if dtype == torch.int8 else
                   (unit.UNIT_F16, unit.unit_matmul_f16, torch.float32))
    es = dtype.itemsize
    # (an operand that is read in place has to be aligned)
    offs = [offset if (k * es) % 16 or (ld * es) % 16 else 0 for ld in (lda, ldb)]
    A, a = matrix(g, dtype, m, k, lda, offs[0])
    B, b = matrix(g, dtype, n, k, ldb, offs[1])
    c = torch.empty((m, n), dtype=out, device=DEV)
    ws = torch.empty(max(unit.unit_matmul_workspace(m, n, k, lda, ldb, ut), 256), dtype=torch.uint8, device=DEV)
    announce("pad rows", dtype, (m, n, k), (lda, ldb), offs)
    fn(m, n, k, A, lda, B, ldb, c, n, ws)
    torch.cuda.synchronize()
    assert torch.equal(c.double(), a.double() @ b.double().t())
