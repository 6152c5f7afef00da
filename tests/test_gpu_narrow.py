"""Convs of at most four input channels (kernels_narrow.hip): both pixel tiles, every operand type, NCHW and packed input, raw and
requantised results, at the edges of tiles, windows and images."""
import numpy as np
import pytest
import torch

import oracle
from paper_2101_08458_amd import unit
from gpu_util import announce

pytestmark = pytest.mark.gpu

# n, c, (h, w), k, (r, s), stride, pad; the last three take 256 pixels a workgroup, the others 64
SHAPES = [
    (1, 3, (32, 32), 64, (7, 7), (2, 2), (3, 3)),
    (2, 1, (9, 4), 33, (3, 3), (1, 1), (1, 1)),
    (1, 4, (5, 13), 65, (1, 1), (1, 1), (0, 0)),
    (2, 2, (11, 17), 96, (5, 4), (1, 2), (2, 1)),
    (1, 3, (8, 70), 16, (8, 8), (3, 1), (0, 5)),
    (3, 3, (7, 6), 40, (2, 5), (2, 3), (4, 7)),
    (12, 3, (97, 131), 130, (7, 7), (2, 2), (3, 3)),
    (9, 4, (40, 75), 200, (3, 3), (1, 1), (0, 0)),
    (20, 1, (64, 64), 64, (4, 6), (1, 1), (1, 2)),
]
TYPES = {"i8": torch.int8, "u8i8": torch.uint8, "f16": torch.float16, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}


def _case(shape, dtype):
    n, c, hw, k, win, stride, pad = shape
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n * hw[1] + k)
    x = torch.randint(0 if dtype == "u8i8" else -4, 5, (n, c) + hw, generator=g, device="cuda:0")
    w = torch.randint(1, 5, (k, c) + win, generator=g, device="cuda:0") * (2 * torch.randint(0, 2, (k, c) + win, generator=g, device="cuda:0") - 1)
    return x, w, unit.conv_desc(n, c, *hw, k, *win, stride, pad)


@pytest.mark.parametrize("dtype", sorted(TYPES))
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_raw_sums(shape, dtype):
    x, w, d = _case(shape, dtype)
    ut, ints = getattr(unit, "UNIT_" + dtype.upper()), dtype in ("i8", "u8i8")
    xd, wd = x.float().to(TYPES[dtype]), w.float().to(torch.int8 if ints else TYPES[dtype])
    x64 = x.double()
    if not ints:            # one pixel that is not finite: only the windows that hold it may see it
        h, v = shape[2][0] // 2, float("nan") if dtype == "fp8" else float("inf")
        xd[0, 0, h, 1], x64[0, 0, h, 1] = v, v
    exact = torch.nn.functional.conv2d(x64, w.double(), stride=shape[5], padding=shape[6])
    ws = torch.empty(unit.unit_conv2d_workspace(d, ut) + 256, dtype=torch.uint8, device="cuda:0")
    fn, results = getattr(unit, "unit_conv2d_" + dtype), {}
    announce("narrow raw", dtype, shape)
    new = lambda: torch.full(exact.shape, -7, device="cuda:0", dtype=torch.int32 if ints else torch.float32)
    y = results["plain"] = new()
    fn(d, xd, wd, y, None, None, ws) if dtype == "i8" else fn(d, xd, wd, y, ws)
    if dtype in ("i8", "f16"):
        wp = torch.empty(unit.unit_packed_weights_bytes(d, ut), dtype=torch.uint8, device="cuda:0")
        xp = torch.empty(unit.unit_packed_act_bytes(shape[0], shape[1], *shape[2], ut), dtype=torch.uint8, device="cuda:0")
        getattr(unit, "unit_pack_weights_" + dtype)(d, wd, wp)
        getattr(unit, "unit_pack_act_" + dtype)(shape[0], shape[1], *shape[2], xd, xp)
        y = results["packed"] = new()
        if dtype == "i8":
            unit.unit_conv2d_packed_i8(d, xp, wp, y, None, None, None, ws)
        else:
            unit.unit_conv2d_packed_f16(d, xp, wp, y, ws)
    torch.cuda.synchronize()
    fine = exact.isfinite()
    for name, y in results.items():
        assert torch.equal(y[fine].double(), exact[fine]), name
        assert not y[~fine].double().isfinite().any(), name


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_requantised(shape, relu):
    x, w, d = _case(shape, "i8")
    acc = torch.nn.functional.conv2d(x.double(), w.double(), stride=shape[5], padding=shape[6]).cpu().numpy().astype(np.int32)
    n, k, p, q = acc.shape
    r = np.random.default_rng(k)
    scale = (0.3 + r.random(k)).astype(np.float32)
    bias = r.integers(-60, 60, k).astype(np.int32)
    exp = oracle.requant(acc, scale, bias=bias, relu=relu)
    dev = lambda t: t.to("cuda:0")
    scale, bias = dev(torch.from_numpy(scale)), dev(torch.from_numpy(bias))
    rq = unit.make_requant(scale, bias, relu=relu)
    xd, wd, kp = x.to(torch.int8), w.to(torch.int8), (k + 15) // 16 * 16
    ws = torch.empty(unit.unit_conv2d_workspace(d, unit.UNIT_I8) + 256, dtype=torch.uint8, device="cuda:0")
    wp = torch.empty(unit.unit_packed_weights_bytes(d, unit.UNIT_I8), dtype=torch.uint8, device="cuda:0")
    xp = torch.empty(unit.unit_packed_act_bytes(n, shape[1], *shape[2], unit.UNIT_I8), dtype=torch.uint8, device="cuda:0")
    y8 = [torch.full(exp.shape, 55, dtype=torch.int8, device="cuda:0") for _ in range(2)]
    yp = [torch.full((n * p * q * kp + 64,), 55, dtype=torch.int8, device="cuda:0") for _ in range(2)]
    announce("narrow requant", shape, relu)
    unit.unit_pack_weights_i8(d, wd, wp)
    unit.unit_pack_act_i8(n, shape[1], *shape[2], xd, xp)
    unit.unit_conv2d_wpacked_i8(d, xd, wp, None, rq, y8[0], ws)
    unit.unit_conv2d_packed_i8(d, xp, wp, None, rq, y8[1], yp[0], ws)       # both results
    unit.unit_conv2d_packed_i8(d, xp, wp, None, rq, None, yp[1], ws)
    torch.cuda.synchronize()
    for y in y8:
        assert np.array_equal(y.cpu().numpy(), exp)
    for y in yp:
        assert (y[n * p * q * kp:] == 55).all(), "past the end"
        got = y[:n * p * q * kp].view(n, p * q, kp).cpu().numpy()
        assert np.array_equal(got[:, :, :k].transpose(0, 2, 1).reshape(exp.shape), exp)
        assert (got[:, :, k:] == 0).all(), "padding channels"
