"""Ends of a reduction in the small tiles' conv modes: last steps that lie past the end in part, slices of a split reduction, fewer steps
than stages; what lies past an end must count as zeros, also where it holds infinities."""
import numpy as np
import pytest
import torch

import oracle
from paper_2101_08458_amd import unit, workloads as wl
from gpu_util import announce, dev, forced, host, same

pytestmark = pytest.mark.gpu

# channels, window, stride, pad: taps of less than a step, whole taps gathered, shifted read, 1x1 read (whole and partial last steps)
CASES = [(24, 3, 1, 1), (128, 3, 2, 1), (256, 3, 1, 1), (256, 1, 1, 0), (100, 1, 1, 0), (40, 1, 1, 0)]


@pytest.mark.parametrize("tile", [2, 3, 4, 5, 9, 12])
@pytest.mark.parametrize("c,win,stride,pad", CASES)
def test_ends_of_the_reduction(c, win, stride, pad, tile):
    g = wl.rng(137, c + win)
    k, hw = 37, 12
    x, w = wl.int8_activations(g, (2, c, hw, hw)), wl.int8_weights(g, (k, c, win, win))
    ref = oracle.conv2d_i8(x, w, (stride, stride), (pad, pad))
    # every other channel's weights are infinite: the channels between them must not see it
    xh, wh = wl.f16_activations(g, (2, c, hw, hw)), wl.f16_weights(g, (k, c, win, win), c * win * win)
    finite = torch.nn.functional.conv2d(dev(xh).view(torch.float16).double(), dev(wh).view(torch.float16).double(), stride=stride, padding=pad)[:, ::2]
    mag = torch.nn.functional.conv2d(dev(xh).view(torch.float16).double().abs(), dev(wh).view(torch.float16).double().abs(), stride=stride, padding=pad)[:, ::2]
    whd = dev(wh).view(torch.float16).clone()
    whd[1::2] = float("inf")
    d = unit.conv_desc(2, c, hw, hw, k, win, win, stride, pad)
    for split in (1, 3):
        announce("slice ends", c, win, stride, pad, "tile", tile, "split", split)
        with forced(tile, split):
            ws = torch.empty(max(unit.unit_conv2d_workspace(d, unit.UNIT_I8), unit.unit_conv2d_workspace(d, unit.UNIT_F16), 256),
                             dtype=torch.uint8, device="cuda:0")
            y = torch.full(ref.shape, -7, dtype=torch.int32, device="cuda:0")
            unit.unit_conv2d_i8(d, dev(x), dev(w), y, None, None, ws)
            yf = torch.full(ref.shape, -7.0, dtype=torch.float32, device="cuda:0")
            unit.unit_conv2d_f16(d, dev(xh), whd, yf, ws)
        torch.cuda.synchronize()
        assert same(host(y), ref, f"int8, split {split}")
        assert ((yf[:, ::2].double() - finite).abs() <= c * win * win * 2.0 ** -24 * mag + 1e-30).all(), f"fp16, split {split}"


# Plain rows whose pitch holds infinities behind the reduction; up to four steps and more than that are kernels of their own.
@pytest.mark.parametrize("tile", [2, 3, 4, 5, 6, 9, 12])
@pytest.mark.parametrize("kbytes", [16, 240, 256, 272, 496, 512, 528, 1024, 1040, 2064])
def test_ends_of_short_products(kbytes, tile):
    m, n, gen = 37, 300, torch.Generator(device="cuda:0")
    gen.manual_seed(kbytes)
    for ut, fn, tt, es in [(unit.UNIT_I8, unit.unit_matmul_i8, torch.int8, 1), (unit.UNIT_U8I8, unit.unit_matmul_u8i8, torch.int8, 1),
                           (unit.UNIT_F16, unit.unit_matmul_f16, torch.float16, 2), (unit.UNIT_BF16, unit.unit_matmul_bf16, torch.bfloat16, 2)]:
        k, ld = kbytes // es, kbytes // es + 32
        if es == 1:
            a = torch.randint(0, 256, (m, ld), generator=gen, device="cuda:0", dtype=torch.uint8)
            a = a if ut == unit.UNIT_U8I8 else a.view(torch.int8)
            b = torch.randint(-128, 128, (n, ld), generator=gen, device="cuda:0", dtype=torch.int8)
        else:
            a, b = (torch.randn((r, ld), generator=gen, device="cuda:0").to(tt) for r in (m, n))
            a[:, k:] = b[:, k:] = float("inf")
        exact = a[:, :k].double() @ b[:, :k].double().t()
        mag = a[:, :k].double().abs() @ b[:, :k].double().abs().t()
        for split in (1, 2):
            announce("short products", ut, (m, n, k), "tile", tile, "split", split)
            with forced(tile, split):
                c = torch.full((m, n), -7, device="cuda:0", dtype=torch.int32 if es == 1 else torch.float32)
                ws = torch.empty(max(unit.unit_matmul_workspace(m, n, k, ld, ld, ut), 256), dtype=torch.uint8, device="cuda:0")
                fn(m, n, k, a, ld, b, ld, c, n, ws)
            torch.cuda.synchronize()
            assert ((c.double() - exact).abs() <= (0 if es == 1 else k * 2.0 ** -24) * mag).all(), (ut, split)
