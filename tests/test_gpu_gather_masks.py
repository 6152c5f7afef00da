"""Gather of packed activations: the tap masks at their limits (31 tap rows over all planes, 31 tap columns; wider windows take the
kernel with a bounds test per tap), padding wider than the window, unpadded windows, planes in the padding.  Pixels of whole steps of
channels (scalar tap walk) and of less (a tap per lane).  Integer sums, bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2101_08458_amd import unit, workloads as wl
from gpu_util import announce, dev, forced, host, same

pytestmark = pytest.mark.gpu

# (d, h, w), (t, r, s), stride, pad
CASES = [((1, 33, 6), (1, 31, 2), (1, 1, 1), (0, 15, 1)), ((1, 34, 5), (1, 32, 1), (1, 1, 1), (0, 16, 0)),
         ((1, 4, 35), (1, 2, 31), (1, 1, 2), (0, 1, 15)), ((1, 3, 34), (1, 1, 32), (1, 1, 1), (0, 0, 16)),
         ((33, 3, 3), (31, 1, 2), (1, 1, 1), (15, 0, 1)), ((7, 9, 8), (5, 6, 3), (1, 2, 1), (2, 3, 1)),
         ((6, 9, 8), (4, 8, 3), (2, 1, 1), (1, 4, 1)), ((1, 5, 4), (1, 3, 3), (1, 2, 1), (0, 5, 4)),
         ((2, 5, 4), (1, 3, 1), (1, 1, 1), (3, 1, 0)), ((3, 8, 7), (2, 3, 3), (1, 2, 1), (0, 0, 0))]


@pytest.mark.parametrize("dims,win,stride,pad", CASES)
@pytest.mark.parametrize("c", [128, 24])
def test_taps_at_the_border(c, dims, win, stride, pad):
    g = wl.rng(130, c + sum(dims))
    x, w = wl.int8_activations(g, (2, c) + dims), wl.int8_weights(g, (20, c) + win)
    ref = oracle.conv3d_i8(x, w, stride, pad)
    d = unit.conv3d_desc(2, c, *dims, 20, *win, stride, pad)
    xd, wd = dev(x), dev(w)
    for tile, split in [(None, None), (3, 2), (4, 1), (1, 1), (8, 1)]:
        announce("tap masks", c, dims, win, stride, pad, "tile", tile, "split", split)
        with forced(tile=tile, split=split):
            ws = torch.empty(max(unit.unit_conv3d_workspace(d, unit.UNIT_I8), 256), dtype=torch.uint8, device="cuda:0")
            y = torch.full(ref.shape, -7, dtype=torch.int32, device="cuda:0")
            unit.unit_conv3d_i8(d, xd, wd, y, ws)
        torch.cuda.synchronize()
        assert same(host(y), ref, f"tile {tile} split {split}")


# One plane of input and one tap plane, with padding in depth: the output planes beside the middle one lie wholly in the padding and
# are zero, whatever the neighbouring images hold.
@pytest.mark.parametrize("c,win,stride,pad", [(128, (1, 3, 3), (1, 2, 2), (1, 1, 1)), (24, (1, 3, 3), (1, 1, 1), (1, 1, 1)),
                                              (40, (1, 1, 1), (1, 2, 2), (1, 0, 0)), (128, (1, 3, 2), (2, 1, 1), (2, 0, 1)),
                                              (24, (1, 5, 3), (3, 2, 1), (2, 2, 1))])
def test_depth_padding_around_one_plane(c, win, stride, pad):
    g = wl.rng(134, c + sum(win))
    x, w = wl.int8_activations(g, (3, c, 1, 8, 9)), wl.int8_weights(g, (20, c) + win)
    ref = oracle.conv3d_i8(x, w, stride, pad)
    d = unit.conv3d_desc(3, c, 1, 8, 9, 20, *win, stride, pad)
    announce("depth padding", c, win, stride, pad)
    ws = torch.empty(max(unit.unit_conv3d_workspace(d, unit.UNIT_I8), 256), dtype=torch.uint8, device="cuda:0")
    y = torch.full(ref.shape, -7, dtype=torch.int32, device="cuda:0")
    unit.unit_conv3d_i8(d, dev(x), dev(w), y, ws)
    torch.cuda.synchronize()
    assert same(host(y), ref, "depth padding")


# Windows too wide for the masks on the large four-wave tiles, which have no kernel for them: those calls run on the eight-wave tiles of
# the same shapes, raw and requantised.
@pytest.mark.parametrize("tile", [14, 15, 16])
@pytest.mark.parametrize("c", [128, 24])
@pytest.mark.parametrize("dims,win,pad", [((34, 9), (32, 1), (16, 0)), ((4, 36), (2, 32), (1, 16)), ((9, 8), (3, 3), (1, 1))])
def test_wide_windows_on_large_tiles(dims, win, pad, c, tile):
    g = wl.rng(138, c + sum(dims))
    n, k = 3, 150
    x, w = wl.int8_activations(g, (n, c) + dims), wl.int8_weights(g, (k, c) + win)
    ref = oracle.conv2d_i8(x, w, (1, 1), pad)
    scale = (127.0 / np.abs(ref).max(axis=(0, 2, 3)).clip(1)).astype(np.float32)
    bytes_ref = oracle.requant(ref, scale, relu=False)
    xh, wh = wl.f16_activations(g, (n, c) + dims), wl.f16_weights(g, (k, c) + win, c * win[0] * win[1])
    d = unit.conv_desc(n, c, *dims, k, *win, 1, pad)
    xd, wd, sd = dev(x), dev(w), dev(scale)
    xhd, whd = dev(xh), dev(wh)
    x64, w64 = xhd.view(torch.float16).double(), whd.view(torch.float16).double()
    exact, mag = (torch.nn.functional.conv2d(a, b, padding=pad) for a, b in ((x64, w64), (x64.abs(), w64.abs())))
    for split in (1, 2):
        announce("wide windows", c, dims, win, "tile", tile, "split", split)
        with forced(tile, split):
            ws = torch.empty(max(unit.unit_conv2d_workspace(d, unit.UNIT_I8), unit.unit_conv2d_workspace(d, unit.UNIT_F16), 256),
                             dtype=torch.uint8, device="cuda:0")
            y = torch.full(ref.shape, -7, dtype=torch.int32, device="cuda:0")
            unit.unit_conv2d_i8(d, xd, wd, y, None, None, ws)
            y8 = torch.full(ref.shape, -7, dtype=torch.int8, device="cuda:0")
            unit.unit_conv2d_i8(d, xd, wd, None, unit.make_requant(sd, relu=False), y8, ws)
            yf = torch.full(ref.shape, -7.0, dtype=torch.float32, device="cuda:0")
            unit.unit_conv2d_f16(d, xhd, whd, yf, ws)
        torch.cuda.synchronize()
        assert same(host(y), ref, f"raw, split {split}")
        assert same(host(y8), bytes_ref, f"requantised, split {split}")
        assert ((yf.double() - exact).abs() <= c * win[0] * win[1] * 2.0 ** -24 * mag + 1e-30).all(), f"fp16, split {split}"
