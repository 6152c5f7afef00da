"""Layout passes: packed weights byte for byte (rows of more and of fewer chunks than a workgroup's threads, partial chunks, one tap),
and plain conv calls, which pack both operands in one launch, on each kind of activation pass (aligned rows, unaligned rows,
subsampled 1x1, channels that fit one chunk) with the weights' sums taken on the way."""
import numpy as np
import pytest
import torch

import oracle
from paper_2101_08458_amd import unit, workloads as wl
from gpu_util import announce, dev, host, same

pytestmark = pytest.mark.gpu


def scratch(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda:0")


@pytest.mark.parametrize("k,c,r", [(5, 512, 3), (3, 17, 7), (7, 255, 1), (2, 9, 5), (1, 4096, 1), (4, 1, 1)])
@pytest.mark.parametrize("dtype", ["i8", "f16"])
def test_packed_weights_bytes(dtype, k, c, r):
    np_t, ut, ch = (np.int8, unit.UNIT_I8, 16) if dtype == "i8" else (np.uint16, unit.UNIT_F16, 8)
    g = wl.rng(132, c)
    w = g.integers(np.iinfo(np_t).min, np.iinfo(np_t).max + 1, (k, c, r, r)).astype(np_t)
    cp = (c + ch - 1) // ch * ch
    exp = np.zeros((k, r, r, cp), np_t)
    exp[..., :c] = w.transpose(0, 2, 3, 1)
    d = unit.conv_desc(1, c, r, r, k, r, r)
    wp = scratch(unit.unit_packed_weights_bytes(d, ut))
    announce("pack weights", dtype, k, c, r)
    (unit.unit_pack_weights_i8 if dtype == "i8" else unit.unit_pack_weights_f16)(d, dev(w), wp)
    torch.cuda.synchronize()
    assert same(host(wp).view(np_t)[:exp.size].reshape(exp.shape), exp, "packed weights")


# n, c, h, w, k, window, stride, pad
CASES = [(2, 512, 8, 8, 19, 3, 1, 1), (2, 40, 7, 7, 33, 3, 1, 1), (3, 96, 9, 11, 20, 1, 2, 0), (2, 3, 20, 18, 24, 7, 2, 3), (1, 13, 9, 9, 18, 3, 1, 0)]


@pytest.mark.parametrize("n,c,h,w_,k,win,stride,pad", CASES)
def test_plain_calls(n, c, h, w_, k, win, stride, pad):
    g = wl.rng(133, c + h)
    w = wl.int8_weights(g, (k, c, win, win))
    d = unit.conv_desc(n, c, h, w_, k, win, win, stride, pad)
    p, q = unit.unit_conv2d_out_dims(d)
    for ut, fn, x in [(unit.UNIT_I8, unit.unit_conv2d_i8, wl.int8_activations(g, (n, c, h, w_))),
                      (unit.UNIT_U8I8, unit.unit_conv2d_u8i8, g.integers(0, 256, (n, c, h, w_)).astype(np.uint8))]:
        ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), stride=stride, padding=pad)
        y = torch.full((n, k, p, q), -7, dtype=torch.int32, device="cuda:0")
        ws = scratch(unit.unit_conv2d_workspace(d, ut))
        announce("plain conv", ut, (n, c, h, w_, k, win, stride, pad))
        if ut == unit.UNIT_I8:
            fn(d, dev(x), dev(w), y, None, None, ws)
        else:
            fn(d, dev(x), dev(w), y, ws)
        torch.cuda.synchronize()
        assert same(host(y), ref.numpy().astype(np.int32), f"type {ut}")


# Pixels of one chunk: a kernel each for up to 4, 8 and 16 channels, with and without weights in the same launch.
@pytest.mark.parametrize("c", [1, 4, 5, 8, 9, 16])
def test_few_channels(c):
    test_plain_calls(2, c, 20, 18, 24, 5, 2, 2)
    g = wl.rng(136, c)
    for dtype, np_t, ch in (("i8", np.int8, 16), ("f16", np.uint16, 8)):
        if c > ch:
            continue
        x = g.integers(np.iinfo(np_t).min, np.iinfo(np_t).max + 1, (3, c, 19, 23)).astype(np_t)
        exp = np.zeros((3, 19, 23, ch), np_t)
        exp[..., :c] = x.transpose(0, 2, 3, 1)
        xp = scratch((exp.nbytes + 255) // 256 * 256)
        announce("pack activations", dtype, c)
        (unit.unit_pack_act_i8 if dtype == "i8" else unit.unit_pack_act_f16)(3, c, 19, 23, dev(x), xp)
        torch.cuda.synchronize()
        assert same(host(xp).view(np_t)[:exp.size].reshape(exp.shape), exp, "packed activations")


# Many output channels of few chunks: several to a workgroup, and the last workgroup partly empty.
@pytest.mark.parametrize("k,c,r", [(100003, 16, 1), (4099, 5, 3), (2051, 33, 1)])
@pytest.mark.parametrize("dtype", ["i8", "f16"])
def test_packed_weights_of_many_channels(dtype, k, c, r):
    test_packed_weights_bytes(dtype, k, c, r)


# Unsigned activations: more output channels than the launch has workgroups for weights (2^20), and images whose packing takes more
# workgroups than a flat grid holds (2^24), so that weights and activations are packed in a launch each.
@pytest.mark.parametrize("n,c,k", [(1, 9, (1 << 20) + 5), (65535, 64 * 256 + 5, 3)])
def test_plain_calls_of_very_many_workgroups(n, c, k):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n + c)
    w = torch.randint(-128, 128, (k, c, 1, 1), generator=g, device="cuda:0", dtype=torch.int8)
    x = torch.randint(0, 256, (n, c, 1, 1), generator=g, device="cuda:0", dtype=torch.uint8)
    d = unit.conv_desc(n, c, 1, 1, k, 1, 1)
    y = torch.full((n, k, 1, 1), -7, dtype=torch.int32, device="cuda:0")
    ws = scratch(unit.unit_conv2d_workspace(d, unit.UNIT_U8I8))
    announce("plain conv, many workgroups", n, c, k)
    unit.unit_conv2d_u8i8(d, x, w, y, ws)
    torch.cuda.synchronize()
    wd = w.view(k, c).double()
    ref = torch.cat([part.double() @ wd.t() for part in x.view(n, c).split(8192)])
    assert torch.equal(y.view(n, k), ref.to(torch.int32))
