"""The requantise epilogue's NCHW bytes: every tile shape, with images whose pixels are whole 16-byte pieces, whole
dwords or neither (pieces that cross from one image into the next), channel counts that end inside a group of four,
and an output that starts on an odd byte.  Bit-exact against the oracle, nothing written outside the output."""
import numpy as np
import pytest
import torch

import oracle
from paper_2101_08458_amd import unit, workloads as wl
from gpu_util import announce, dev, host, forced, same

pytestmark = pytest.mark.gpu

# (images, channels in, height, width, channels out)
SHAPES = [(3, 32, 8, 8, 70), (5, 48, 6, 6, 33), (5, 32, 7, 7, 130), (7, 16, 1, 3, 36), (2, 16, 1, 1, 5), (1, 64, 17, 19, 257)]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n,c,h,w,k", SHAPES)
def test_requant_nchw_bytes_all_tiles(n, c, h, w, k, shift):
    x, wt = wl.conv_inputs_i8(wl.conv_shape(c, h, k, 1, 1, 0), n, 11)
    x = np.resize(x, (n, c, h, w))
    acc = oracle.conv2d_i8(x, wt, (1, 1), (0, 0))
    bias = np.random.default_rng(5).integers(-900, 900, k).astype(np.int32)
    scale = (127.0 / np.abs(acc).max(axis=(0, 2, 3)).clip(1)).astype(np.float32)
    exp = oracle.requant(acc, scale, bias=bias, relu=False)
    d = unit.conv_desc(n, c, h, w, k, 1, 1, 1, 0)
    xd, wd, sd, bd = dev(x), dev(wt), dev(scale), dev(bias)
    wp = torch.empty(unit.unit_packed_weights_bytes(d, unit.UNIT_I8), dtype=torch.uint8, device="cuda:0")
    unit.unit_pack_weights_i8(d, wd, wp)
    rq = unit.make_requant(sd, bd, relu=False)
    size = exp.size
    for tile in (None, *range(13)):
        with forced(tile, 1 if tile is not None else None):
            ws = torch.empty(max(unit.unit_conv2d_wpacked_workspace(d, unit.UNIT_I8), 256), dtype=torch.uint8, device="cuda:0")
            buf = torch.full((size + 64,), -77, dtype=torch.int8, device="cuda:0")
            announce("requant rows", (n, c, h, w, k), "shift", shift, "tile", tile)
            unit.unit_conv2d_wpacked_i8(d, xd, wp, None, rq, buf[16 + shift:16 + shift + size], ws)
            torch.cuda.synchronize()
        got = host(buf)
        assert same(got[16 + shift:16 + shift + size].reshape(exp.shape), exp, f"tile {tile}")
        assert (got[:16 + shift] == -77).all() and (got[16 + shift + size:] == -77).all(), f"tile {tile}: written outside"
