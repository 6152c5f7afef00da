"""128x128 tile with four LDS stages: ring start-up and remainders of the unrolled step loop (fewer steps than stages, one more,
a last step that is partly empty), rows and columns that end inside a tile, a split reduction, every operand type.  Integer sums bit-exact; 16-bit float sums against fp64 within a few fp32 roundings of the sum of magnitudes,
fp8 within the bits its matrix instruction keeps."""
import pytest
import torch

from paper_2101_08458_amd import unit
from gpu_util import announce, chosen_tile, forced

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TILE = 13
FNS = {"i8": (unit.UNIT_I8, unit.unit_matmul_i8), "u8i8": (unit.UNIT_U8I8, unit.unit_matmul_u8i8),
       "f16": (unit.UNIT_F16, unit.unit_matmul_f16), "bf16": (unit.UNIT_BF16, unit.unit_matmul_bf16),
       "fp8": (unit.UNIT_FP8, unit.unit_matmul_fp8)}
TT = {"f16": torch.float16, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}


def operand(g, dtype, shape, first):
    if dtype in ("i8", "u8i8"):
        if first and dtype == "u8i8":
            return torch.randint(0, 256, shape, generator=g, device=DEV, dtype=torch.uint8)
        return torch.randint(-128, 128, shape, generator=g, device=DEV, dtype=torch.int8)
    return torch.randn(shape, generator=g, device=DEV).to(TT[dtype])


def check(got, a, b, dtype):
    exact = a.double() @ b.double().t()
    if dtype in ("i8", "u8i8"):
        assert torch.equal(got.double(), exact)
        return
    mag = a.double().abs() @ b.double().abs().t()
    # K roundings of 2^-24 at worst, sqrt(K) in practice; the fp8 instruction keeps fewer bits of a group of products
    bound = 1e-4 if dtype == "fp8" else a.shape[1] * 2.0 ** -24
    assert ((got.double() - exact).abs() <= bound * mag + 1e-30).all()


@pytest.mark.parametrize("dtype", sorted(FNS))
def test_matmul_steps_and_edges(dtype):
    ut, fn = FNS[dtype]
    es = 2 if dtype in ("f16", "bf16") else 1
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    for m, n, kbytes, split in [(128, 128, 128, 1), (20, 30, 16, 1), (129, 257, 3 * 128 + 16, 1), (200, 100, 4 * 128, 1),
                                (130, 126, 5 * 128 - 48, 1), (255, 129, 11 * 128 + 32, 2), (64, 300, 9 * 128, 3), (100, 77, 777, 1)]:
        k = kbytes // es
        a, b = operand(g, dtype, (m, k), True), operand(g, dtype, (n, k), False)
        c = torch.empty((m, n), device=DEV, dtype=torch.int32 if dtype in ("i8", "u8i8") else torch.float32)
        with forced(TILE, split):
            ws = torch.empty(max(unit.unit_matmul_workspace(m, n, k, k, k, ut), 256), dtype=torch.uint8, device=DEV)
            announce("deep ring matmul", dtype, (m, n, k), "split", split)
            fn(m, n, k, a, k, b, k, c, n, ws)
        torch.cuda.synchronize()
        check(c, a, b, dtype)


# by the rule, not forced: several bands of eight row tiles with columns that end inside a tile (B of more than 8 MiB: the
# banded tile order; less: runs along a row tile), row pitch of C beyond its width, tiles with half of their rows empty
BY_RULE = [(1533, 2001, 4224, 37), (2048, 2048, 272, 0), (129, 12000, 400, 3), (16500, 65, 160, 64), (1100, 1900, 130, 1)]


@pytest.mark.parametrize("m,n,k,extra", BY_RULE)
@pytest.mark.parametrize("dtype", sorted(FNS))
def test_matmul_chosen_by_the_rule(dtype, m, n, k, extra):
    ut, fn = FNS[dtype]
    es = 2 if dtype in ("f16", "bf16") else 1
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    assert chosen_tile(m, n, -(-k * es // 16), ut) == TILE
    a, b = operand(g, dtype, (m, k), True), operand(g, dtype, (n, k), False)
    ldc = n + extra
    poison = -77 if dtype in ("i8", "u8i8") else float("nan")
    c = torch.full((m + 1, ldc), poison, device=DEV, dtype=torch.int32 if dtype in ("i8", "u8i8") else torch.float32)
    ws = torch.empty(max(unit.unit_matmul_workspace(m, n, k, k, k, ut), 256), dtype=torch.uint8, device=DEV)
    announce("deep ring matmul by the rule", dtype, (m, n, k), "pitch", ldc)
    fn(m, n, k, a, k, b, k, c, ldc, ws)
    torch.cuda.synchronize()
    check(c[:m, :n], a, b, dtype)
    untouched = torch.cat([c[:m, n:].reshape(-1), c[m]])
    assert (untouched == -77).all() if dtype in ("i8", "u8i8") else untouched.isnan().all()
