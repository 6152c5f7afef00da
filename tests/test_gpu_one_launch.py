"""Products of several rounds of large tiles that run as one launch of a narrower tile (or of the large one) in place of two column
ranges: the choice, and every element, with rows and columns that end inside a tile."""
import pytest
import torch

from paper_2101_08458_amd import unit
from gpu_util import announce

pytestmark = pytest.mark.gpu
TYPES = {"i8": torch.int8, "f16": torch.float16, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}


@pytest.mark.parametrize("dtype", sorted(TYPES))
@pytest.mark.parametrize("m,n,chunks", [(4801, 6700, 56), (3136, 7424, 64), (3200, 4929, 96), (6720, 6336, 32)])
def test_products(m, n, chunks, dtype):
    if chunks == 32 and dtype == "fp8":
        pytest.skip("two ranges in the type without four-wave tiles")
    ints, ut, k = dtype == "i8", getattr(unit, "UNIT_" + dtype.upper()), chunks * 16 // (2 if dtype in ("f16", "bf16") else 1)
    info = unit.unit_select_matmul(m, n, k, ut)
    assert (info.block_m, info.split_k, info.tail_block_n) == (256, 1, 0) and info.workgroups == -(-m // 256) * -(-n // info.block_n) > 256
    assert info.block_n in ((256,) if chunks == 32 else (128, 192))
    g = torch.Generator(device="cuda:0")
    g.manual_seed(m)
    a = torch.randint(-3, 4, (m, k), generator=g, device="cuda:0")
    b = torch.randint(-3, 4, (n, k), generator=g, device="cuda:0")        # (small integers: exact in every type and order)
    exact = a.float() @ b.float().t()                                     # (below 2^24)
    a, b = a.float().to(TYPES[dtype]), b.float().to(TYPES[dtype])
    c = torch.full((m, n + 5), -7, device="cuda:0", dtype=torch.int32 if ints else torch.float32)
    ws = torch.empty(unit.unit_matmul_workspace(m, n, k, k, k, ut) + 256, dtype=torch.uint8, device="cuda:0")
    announce("one launch", dtype, (m, n, k))
    getattr(unit, "unit_matmul_" + dtype)(m, n, k, a, k, b, k, c, n + 5, ws)
    torch.cuda.synchronize()
    assert torch.equal(c[:, :n].float(), exact) and (c[:, n:] == -7).all()
