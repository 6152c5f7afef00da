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


# Products of at most 16 rows once ran on 16x64 tiles (index 5) whose reduction was split across workgroups by the rule: their error
# against 64 bits is the measure.  (5 %: the rms over 16000 outputs of either side scatters by less than 1 %.)
@pytest.mark.parametrize("k", [1024, 2304, 2560, 3000, 3072, 4096, 8000])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_error_no_larger_than_of_a_split_reduction(dtype, k):
    ut, fn, tt = FNS[dtype]
    m, n = 16, 4096
    assert chosen_tile(m, n, k // 8, ut) in (12, 17)
    g = torch.Generator(device=DEV)
    g.manual_seed(k)
    a, b = torch.randn((m, k), generator=g, device=DEV).to(tt), torch.randn((n, k), generator=g, device=DEV).to(tt)
    exact, err = a.double() @ b.double().t(), {}
    for tile in (None, 5):
        announce("error of few rows", dtype, (m, n, k), "tile", tile)
        with forced(tile):
            c = torch.empty((m, n), device=DEV)
            ws = torch.empty(max(unit.unit_matmul_workspace(m, n, k, k, k, ut), 256), dtype=torch.uint8, device=DEV)
            fn(m, n, k, a, k, b, k, c, n, ws)
        torch.cuda.synchronize()
        err[tile] = float((c.double() - exact).norm() / exact.norm())
    assert err[None] <= 1.05 * err[5], err
