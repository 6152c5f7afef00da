"""Products of few rows: 16x16 tiles with 256- and 512-byte steps, where the rule puts them and forced: a reduction that ends inside a
step, fewer steps than stages, columns that end inside a tile, row pitches, one row.  Integer sums bit-exact; 16-bit float sums
within K fp32 roundings of the sum of magnitudes."""
import pytest
import torch

from paper_2101_08458_amd import unit
from gpu_util import announce, chosen_tile, forced

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FNS = {"i8": (unit.UNIT_I8, unit.unit_matmul_i8, torch.int8), "u8i8": (unit.UNIT_U8I8, unit.unit_matmul_u8i8, torch.int8),
       "f16": (unit.UNIT_F16, unit.unit_matmul_f16, torch.float16), "bf16": (unit.UNIT_BF16, unit.unit_matmul_bf16, torch.bfloat16)}
# rows, columns, reduction bytes, tile by the rule (None: forced 17)
CASES = [(5, 100, 512, 12), (16, 8192, 1040, 12), (9, 70, 383 * 16, 12), (16, 77, 384 * 16, 17), (7, 4100, 1000 * 16, 17), (7, 600, 1000 * 16, 5),
         (6, 8208, 512, 5), (33, 300, 400 * 16, 17), (17, 2000, 1023 * 16, 17), (17, 50, 1024 * 16, 12), (1, 33, 6160, 17),
         (20, 30, 16, None), (40, 17, 512 * 3 + 48, None), (16, 16, 512 * 5, None)]


@pytest.mark.parametrize("m,n,kbytes,tile", CASES)
@pytest.mark.parametrize("dtype", sorted(FNS))
def test_few_rows(dtype, m, n, kbytes, tile):
    ut, fn, tt = FNS[dtype]
    whole = "i8" in dtype
    k = kbytes if whole else kbytes // 2
    if tile is not None:
        assert chosen_tile(m, n, -(-kbytes // 16), ut) == tile
    g = torch.Generator(device=DEV)
    g.manual_seed(m + n + k)
    ld = k + 64
    if whole:
        a = torch.randint(0, 256, (m, ld), generator=g, device=DEV, dtype=torch.uint8)
        a = a if dtype == "u8i8" else a.view(torch.int8)
        b = torch.randint(-128, 128, (n, ld), generator=g, device=DEV, dtype=torch.int8)
    else:
        a, b = torch.randn((m, ld), generator=g, device=DEV).to(tt), torch.randn((n, ld), generator=g, device=DEV).to(tt)
    c = torch.full((m + 1, n + 3), -77, device=DEV, dtype=torch.int32 if whole else torch.float32)
    announce("few rows", dtype, (m, n, k), "tile", tile)
    with forced(17 if tile is None else None, 1 if tile is None else None):
        ws = torch.empty(max(unit.unit_matmul_workspace(m, n, k, ld, ld, ut), 256), dtype=torch.uint8, device=DEV)
        fn(m, n, k, a, ld, b, ld, c, n + 3, ws)
    torch.cuda.synchronize()
    a, b, got = a[:, :k].double(), b[:, :k].double(), c[:m, :n].double()
    if whole:
        assert torch.equal(got, a @ b.t())
    else:
        assert ((got - a @ b.t()).abs() <= k * 2.0 ** -24 * (a.abs() @ b.abs().t()) + 1e-30).all()
    assert (c[:m, n:] == -77).all() and (c[m] == -77).all()
