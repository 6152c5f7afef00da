"""The rule that gives a plain product the 128x128 tile with four LDS stages, at each of its bounds (host arithmetic)."""
import os

import pytest

from paper_2101_08458_amd import unit
from gpu_util import chosen_tile

TWO_STAGE, FOUR_STAGE, TILE_64 = 1, 13, 3
TYPES = [unit.UNIT_I8, unit.UNIT_F16, unit.UNIT_BF16, unit.UNIT_U8I8, unit.UNIT_FP8]


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(unit.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()


@pytest.mark.parametrize("dtype", TYPES)
def test_bounds(dtype):
    t = lambda m, n, chunks=64: chosen_tile(m, n, chunks, dtype)
    # 16 x 32 tiles of 64x64 are one round of two workgroups per unit, one column more starts the second
    assert t(1024, 2048) != FOUR_STAGE and t(1024, 2049) == FOUR_STAGE
    # 16 x 16 tiles of 128x128 are one per unit, one column or row more is beyond
    assert t(2048, 2048) == FOUR_STAGE and t(2048, 2049) != FOUR_STAGE and t(2049, 2048) != FOUR_STAGE
    # half-empty tiles too; 64 rows or fewer never (513 tiles of 64 columns are 257 of 128)
    assert t(65, 32768) == FOUR_STAGE and t(130, 16384) == FOUR_STAGE and t(16000, 129) == FOUR_STAGE
    assert all(t(64, n) != FOUR_STAGE for n in (16448, 32768, 32769, 65536))


@pytest.mark.parametrize("dtype", TYPES)
def test_one_step_keeps_the_two_stage_tile(dtype):
    t = lambda m, n, chunks: chosen_tile(m, n, chunks, dtype)
    for m, n in [(2048, 2048), (2000, 1900), (4000, 1000), (8192, 257), (128, 32768)]:
        assert t(m, n, 1) == TWO_STAGE and t(m, n, 8) == TWO_STAGE and t(m, n, 9) == FOUR_STAGE
    # ... where it was the choice: not in place of 64x64 tiles
    for m, n in [(1664, 1664), (65, 20000), (384, 5504)]:
        assert t(m, n, 1) == FOUR_STAGE and t(m, n, 8) == FOUR_STAGE


def test_convolution_input_never():
    for bsrc in (1, 2, 3):
        for dtype in (unit.UNIT_I8, unit.UNIT_F16):
            assert all(chosen_tile(k, px, chunks, dtype, bsrc) != FOUR_STAGE
                       for k, px, chunks in [(1024, 3136, 16), (512, 4096, 64), (256, 12544, 72)])
