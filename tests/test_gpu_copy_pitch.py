"""Unaligned matmul operands: their copies have whole 128-byte lines per row where the workspace has room for that, and the bare 16-byte
multiple in a workspace of just that size; one byte less is refused.  Reductions around a line and around 4 KiB."""
import pytest
import torch

from paper_2101_08458_amd import unit
from gpu_util import announce

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def up(v, a):
    return (v + a - 1) // a * a


@pytest.mark.parametrize("m,n,k,lda,ldb", [(33, 70, 127, 127, 127), (5, 300, 129, 144, 131), (140, 90, 4095, 4095, 4099), (300, 257, 4081, 4081, 4096),
                                          (2, 40, 1000, 1001, 1008)])
@pytest.mark.parametrize("dtype", ["i8", "u8i8"])
def test_both_pitches(dtype, m, n, k, lda, ldb):
    ut, fn = (unit.UNIT_I8, unit.unit_matmul_i8) if dtype == "i8" else (unit.UNIT_U8I8, unit.unit_matmul_u8i8)
    g = torch.Generator(device=DEV)
    g.manual_seed(k)
    a = torch.randint(0, 256, (m, lda), generator=g, device=DEV, dtype=torch.uint8)
    a = a if dtype == "u8i8" else a.view(torch.int8)
    b = torch.randint(-128, 128, (n, ldb), generator=g, device=DEV, dtype=torch.int8)
    exact = a[:, :k].double() @ b[:, :k].double().t()
    full = unit.unit_matmul_workspace(m, n, k, lda, ldb, ut)
    pad = lambda rows, ld: up(rows * up(k, 16), 256) if k % 16 or ld % 16 else 0
    wide = lambda rows, ld: up(rows * (up(k, 128) + (128 if up(k, 128) % 4096 == 0 else 0)), 256) if k % 16 or ld % 16 else 0
    bare = full - wide(m, lda) - wide(n, ldb) + pad(m, lda) + pad(n, ldb)
    assert 0 < bare <= full
    for size in (full, bare):
        c = torch.full((m, n), -7, dtype=torch.int32, device=DEV)
        announce("copy pitch", dtype, (m, n, k, lda, ldb), "workspace", size, "of", full)
        fn(m, n, k, a, lda, b, ldb, c, n, torch.empty(size, dtype=torch.uint8, device=DEV))
        torch.cuda.synchronize()
        assert torch.equal(c.double(), exact)
    with pytest.raises(unit.UnitError):
        fn(m, n, k, a, lda, b, ldb, c, n, torch.empty(bare - 1, dtype=torch.uint8, device=DEV))


# Rows around the 512 bytes from which copies have whole lines, on tiles of each size and on the one-row kernel.
@pytest.mark.parametrize("m,n", [(2, 70), (40, 150), (600, 513), (2100, 1100)])
@pytest.mark.parametrize("k", [13, 479, 497, 511, 513])
def test_short_rows(k, m, n):
    test_both_pitches("i8", m, n, k, k, k + 3)
