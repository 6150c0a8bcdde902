"""The build's scan of the generated code for a matrix instruction's result that is read too early
(no GPU, text only).  What the compiler itself once wrote for the sums of the fp32 GEMM, and what a
compiler could make of the explicit wait if nothing held it in its place."""
import pytest

from paper_2602_05754_amd.build import mfma_hazards

MFMA = "v_mfma_f32_16x16x4_f32 v[60:63], v17, v51, v[60:63]"
READ = "v_add_f32_e32 v44, v63, v26"
WAIT = "s_nop 15"


def found(*lines):
    return [ins for _, _, ins in mfma_hazards("kernel_a:\n" + "\n".join(lines) + "\ns_endpgm\n")]


def test_waits_and_barriers_are_no_wait_states():
    assert found(MFMA, "s_waitcnt lgkmcnt(0)", "s_barrier", "s_nop 7", READ) == [READ]
    assert found(MFMA, "s_waitcnt lgkmcnt(0)", "s_barrier", "s_nop 9", READ) == []


def test_the_wait_has_to_lie_between():
    assert found(MFMA, WAIT, READ) == []
    assert found(MFMA, READ, WAIT) == [READ]
    assert found(WAIT, MFMA, "v_mov_b32_e32 v1, v2", READ) == [READ]
    assert found(MFMA, WAIT, MFMA, READ) == [READ]
    assert found(MFMA, "ds_write_b128 v69, v[60:63] offset:16") == ["ds_write_b128 v69, v[60:63] offset:16"]
    assert found(MFMA, "v_mov_b32_e32 v63, v1", READ) == []                     # written anew in between


@pytest.mark.parametrize("op,states", [("v_mfma_f32_16x16x32_bf16", 8), ("v_mfma_f32_16x16x4_f32", 10), ("v_mfma_f64_16x16x4_f64", 18)])
def test_every_instruction_has_its_own_number_of_states(op, states):
    lines = f"{op} v[0:7], v[8:9], v[10:11], v[0:7]", "v_mov_b32_e32 v20, v3"
    assert found(lines[0], f"s_nop {states - 1}", lines[1]) == []
    assert found(lines[0], f"s_nop {states - 2}", lines[1]) == [lines[1]]


def test_paths_through_branches_and_loops_are_followed():
    loop = (".LBB0_1:", READ, WAIT, MFMA, "s_cbranch_scc1 .LBB0_1")             # only the second time round
    assert found(*loop) == [READ]
    assert found(".LBB0_1:", READ, MFMA, WAIT, "s_cbranch_scc1 .LBB0_1") == []
    assert found(MFMA, "s_cbranch_scc1 .LBB0_3", WAIT, "s_branch .LBB0_4", ".LBB0_3:", "v_mov_b32_e32 v1, v2", ".LBB0_4:", READ) == [READ]
    assert found(MFMA, "s_branch .LBB0_4", ".LBB0_3:", READ, ".LBB0_4:", "v_mov_b32_e32 v1, v2") == []
