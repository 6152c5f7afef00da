"""Raw sums stored past the L2 (images of whole 64-byte pieces) and through it (any other image, partial sums): every element arrives."""
import pytest
import torch

from paper_2101_08458_amd import unit
from gpu_util import announce, forced

pytestmark = pytest.mark.gpu

# image sides: 16, 48 and 784 pixels are whole pieces, 15, 49 and 783 are not
SIDES = [(4, 4), (6, 8), (28, 28), (3, 5), (7, 7), (27, 29)]


@pytest.mark.parametrize("dtype", ["i8", "f16", "bf16", "fp8", "u8i8"])
@pytest.mark.parametrize("h,w", SIDES)
def test_raw_sums(h, w, dtype):
    n, c, k = 2, 64, 97
    ut = getattr(unit, "UNIT_" + dtype.upper())
    g = torch.Generator(device="cuda:0")
    g.manual_seed(h * w)
    # (small integers: exact in every operand type, and so are their sums)
    for win, pad in ((1, 0), (3, 1)):
        x = torch.randint(0 if dtype == "u8i8" else -4, 5, (n, c, h, w), generator=g, device="cuda:0")
        wt = torch.randint(-4, 5, (k, c, win, win), generator=g, device="cuda:0")
        exact = torch.nn.functional.conv2d(x.double(), wt.double(), padding=pad)
        tt = {"i8": torch.int8, "u8i8": torch.uint8, "f16": torch.float16, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}[dtype]
        xd, wd = x.to(torch.float32).to(tt), wt.to(torch.float32).to(torch.int8 if dtype == "u8i8" else tt)
        d = unit.conv_desc(n, c, h, w, k, win, win, 1, pad)
        for tile, split in ((None, None), (1, 1), (3, 1), (4, 2)):
            announce("raw sums", dtype, (h, w), "window", win, "tile", tile, "split", split)
            with forced(tile, split):
                ws = torch.empty(unit.unit_conv2d_workspace(d, ut) + 256, dtype=torch.uint8, device="cuda:0")
                y = torch.full(exact.shape, -7, device="cuda:0", dtype=torch.int32 if dtype in ("i8", "u8i8") else torch.float32)
                fn = getattr(unit, "unit_conv2d_" + dtype)
                fn(d, xd, wd, y, None, None, ws) if dtype == "i8" else fn(d, xd, wd, y, ws)
            torch.cuda.synchronize()
            assert torch.equal(y.double(), exact), (win, tile, split)
