"""The build's check of inline-assembly MFMAs: a vector write of an operand just before one is found, also around a loop."""
import importlib.util
import os

import pytest

PATH = os.path.join(os.path.dirname(__file__), "..", "paper_2101_08458_amd", "csrc", "check_resources.py")
spec = importlib.util.spec_from_file_location("check_resources", PATH)
check = importlib.util.module_from_spec(spec)
spec.loader.exec_module(check)

MFMA = ("v_mfma_f32_16x16x32_f16", " a[0:3], v[4:7], v[8:11], a[0:3]")


def code(*insts):
    return [(4 * i, op, operands) for i, (op, operands) in enumerate(insts)]


@pytest.mark.parametrize("insts,found", [
    ([("v_mov_b32_e32", " v4, v1"), MFMA], 1), ([("v_mov_b32_e32", " v4, v1"), ("s_nop", " 1"), MFMA], 1),
    ([("v_mov_b32_e32", " v4, v1"), ("s_nop", " 3"), MFMA], 0), ([("v_mov_b32_e32", " v12, v4"), MFMA], 0),
    ([("v_accvgpr_write_b32", " a3, 0"), MFMA], 1), ([MFMA, MFMA], 0), ([("ds_read_b128", " v[4:7], v1"), MFMA], 0),
    # the write stands behind the MFMA, and a branch leads back to it
    ([MFMA, ("v_mov_b32_e32", " v9, v1"), ("s_cbranch_scc1", " 65533")], 1),
    ([MFMA, ("v_mov_b32_e32", " v9, v1"), ("s_nop", " 4"), ("s_cbranch_scc1", " 65532")], 0)])
def test_late_operand_writes(insts, found):
    assert len(check.late_writes(code(*insts))) == found
