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


# (layer, images, first column of the second launch, images to compare): pixels per image a whole number of 16-byte pieces and not
TWO_RANGES = [(wl.LARGE_CONV, 32, 65536, (0, 19, 20, 21, 31)), (wl.ConvShape(512, 57, 57, 256, 1, 1, 1, 0), 32, 65536, (0, 19, 20, 21, 31))]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("sh,n,seam,imgs", TWO_RANGES)
def test_requant_nchw_bytes_two_column_ranges(sh, n, seam, imgs, shift):
    """The same bytes where a layer runs as two launches (256x256 tiles, then 256x192 ones from a column inside image
    20): whole images on both sides of the seam, the first and the last, and nothing outside the output."""
    d = unit.conv_desc(n, sh.c, sh.h, sh.w, sh.k, sh.r, sh.s, sh.stride, sh.pad)
    info = unit.unit_select_conv2d(d, unit.UNIT_I8)
    assert (info.block_n, info.tail_block_n, info.tail_first_col) == (256, 192, seam) and seam // (sh.h * sh.w) == 20
    x, w = wl.conv_inputs_i8(sh, n, 9, 0)
    acc = oracle.conv2d_i8(np.ascontiguousarray(x[list(imgs)]), w, (sh.stride,) * 2, (sh.pad,) * 2)
    bias = np.random.default_rng(6).integers(-9000, 9000, sh.k).astype(np.int32)
    scale = (127.0 / np.abs(acc).max(axis=(0, 2, 3)).clip(1)).astype(np.float32)
    exp = oracle.requant(acc, scale, bias=bias, relu=True)
    xd, wd, sd, bd = dev(x), dev(w), dev(scale), dev(bias)
    wp = torch.empty(unit.unit_packed_weights_bytes(d, unit.UNIT_I8), dtype=torch.uint8, device="cuda:0")
    unit.unit_pack_weights_i8(d, wd, wp)
    rq = unit.make_requant(sd, bd, relu=True)
    ws = torch.empty(unit.unit_conv2d_wpacked_workspace(d, unit.UNIT_I8), dtype=torch.uint8, device="cuda:0")
    size = n * sh.k * sh.h * sh.w
    buf = torch.full((size + 64,), -77, dtype=torch.int8, device="cuda:0")
    announce("requant rows, two ranges", tuple(sh), n, "shift", shift)
    unit.unit_conv2d_wpacked_i8(d, xd, wp, None, rq, buf[16 + shift:16 + shift + size], ws)
    torch.cuda.synchronize()
    got = host(buf)
    y = got[16 + shift:16 + shift + size].reshape(n, sh.k, sh.h, sh.w)
    for i, img in enumerate(imgs):
        assert same(y[img], exp[i], f"image {img}")
    assert (got[:16 + shift] == -77).all() and (got[16 + shift + size:] == -77).all()


@pytest.mark.parametrize("k", [5, 33, 70, 130])
def test_requant_scale_and_bias_are_slices(k):
    """Scale and bias as slices of longer vectors (4-byte aligned only), their neighbours poisoned: every tile, channel
    counts that end inside a group of four, with the raw, the NCHW and the packed output of one call.  A channel that
    took a neighbour's scale would show in its bytes, or in the packed output's padding channels, which are zero."""
    n, c, h = 3, 32, 7
    sh = wl.conv_shape(c, h, k, 1, 1, 0)
    x, wt = wl.conv_inputs_i8(sh, n, 12)
    acc = oracle.conv2d_i8(x, wt, (1, 1), (0, 0))
    bias = np.random.default_rng(7).integers(-900, 900, k).astype(np.int32)
    scale = (127.0 / np.abs(acc).max(axis=(0, 2, 3)).clip(1)).astype(np.float32)
    exp = oracle.requant(acc, scale, bias=bias, relu=False)
    kp = (k + 15) // 16 * 16
    exp_packed = np.zeros((n, h, h, kp), np.int8)
    exp_packed[..., :k] = exp.transpose(0, 2, 3, 1)
    d = unit.conv_desc(n, c, h, h, k, 1, 1, 1, 0)
    u8 = lambda size: torch.empty(max(size, 256), dtype=torch.uint8, device="cuda:0")
    wp, xp = u8(unit.unit_packed_weights_bytes(d, unit.UNIT_I8)), u8(unit.unit_packed_act_bytes(n, c, h, h, unit.UNIT_I8))
    unit.unit_pack_weights_i8(d, dev(wt), wp)
    unit.unit_pack_act_i8(n, c, h, h, dev(x), xp)
    for off in (1, 2, 3):
        sv = torch.full((k + 16,), 1e6, dtype=torch.float32, device="cuda:0")
        bv = torch.full((k + 16,), 1 << 29, dtype=torch.int32, device="cuda:0")
        sv[off:off + k] = dev(scale)
        bv[off:off + k] = dev(bias)
        rq = unit.make_requant(sv[off:off + k], bv[off:off + k], relu=False)
        for tile in (None, *range(13)):
            with forced(tile, 1 if tile is not None else None):
                ws = u8(unit.unit_conv2d_packed_workspace(d, unit.UNIT_I8))
                y32 = torch.full(exp.shape, -7, dtype=torch.int32, device="cuda:0")
                y8 = torch.full(exp.shape, -77, dtype=torch.int8, device="cuda:0")
                yp = torch.full((exp_packed.size + 64,), 99, dtype=torch.int8, device="cuda:0")
                announce("requant scale slices, channels", k, "offset", off, "tile", tile)
                unit.unit_conv2d_packed_i8(d, xp, wp, y32, rq, y8, yp, ws)
                torch.cuda.synchronize()
            assert same(host(y32), acc, f"raw, tile {tile}") and same(host(y8), exp, f"NCHW, tile {tile}")
            p = host(yp)
            assert same(p[:exp_packed.size].reshape(exp_packed.shape), exp_packed, f"packed, tile {tile}")
            assert (p[exp_packed.size:] == 99).all(), f"tile {tile}: written outside"


# The four-wave tiles hand requantised results of short reductions to the eight-wave ones: reductions on both sides of the line (144 chunks
# of 16 bytes for layers of one round of workgroups), channels of whole steps and of less, bytes in both layouts.
@pytest.mark.parametrize("tile", [14, 15, 16])
@pytest.mark.parametrize("c", [240, 256, 272])
def test_requant_on_large_tiles_around_the_line(c, tile):
    n, h, w_, k = 2, 11, 13, 270
    g = wl.rng(139, c)
    x, wt = wl.int8_activations(g, (n, c, h, w_)), wl.int8_weights(g, (k, c, 3, 3))
    acc = oracle.conv2d_i8(x, wt, (1, 1), (1, 1))
    bias = g.integers(-9000, 9000, k).astype(np.int32)
    scale = (127.0 / np.abs(acc).max(axis=(0, 2, 3)).clip(1)).astype(np.float32)
    exp = oracle.requant(acc, scale, bias=bias, relu=True)
    d = unit.conv_desc(n, c, h, w_, k, 3, 3, 1, 1)
    xd, wd, sd, bd = dev(x), dev(wt), dev(scale), dev(bias)
    wp = torch.empty(unit.unit_packed_weights_bytes(d, unit.UNIT_I8), dtype=torch.uint8, device="cuda:0")
    unit.unit_pack_weights_i8(d, wd, wp)
    rq = unit.make_requant(sd, bd, relu=True)
    with forced(tile, 1):
        ws = torch.empty(max(unit.unit_conv2d_wpacked_workspace(d, unit.UNIT_I8), 256), dtype=torch.uint8, device="cuda:0")
        raw = torch.full(acc.shape, -7, dtype=torch.int32, device="cuda:0")
        y8 = torch.full(exp.shape, -7, dtype=torch.int8, device="cuda:0")
        announce("requant around the line", c, "tile", tile)
        unit.unit_conv2d_wpacked_i8(d, xd, wp, raw, rq, y8, ws)
        torch.cuda.synchronize()
    assert same(host(raw), acc, "raw") and same(host(y8), exp, "bytes")
