"""The check of generated assembly (asm_check) on small listings: each hazard it stands for is found, on the straight path
and around a loop, and the same code with the wait states in place passes."""
import pytest

from paper_2306_11975_amd import asm_check

MFMA = "v_mfma_i32_16x16x64_i8 a[0:3], v[0:3], v[4:7], a[0:3]"
LOAD = "global_load_lds_dwordx4 v9, s[6:7]"


def reasons(*body):
    lines = ["kernel:"] + list(body) + ["s_endpgm", ".Lfunc_end0:"]
    return [x.split(": ")[1] for x in asm_check.hazards(lines)]


def filler(n):
    return [f"s_nop {n - 1}"] if n else []


@pytest.mark.parametrize("touch", ["v_accvgpr_read_b32 v20, a3", "v_accvgpr_mov_b32 a80, a0", "scratch_store_dwordx4 off, a[0:3], s0"])
def test_accumulators_behind_an_mfma(touch):
    assert reasons(MFMA, *filler(11), touch) == ["an accumulation register is touched behind an MFMA"]
    assert reasons(MFMA, *filler(12), touch) == []
    assert reasons(MFMA, "s_add_u32 s0, s0, 1", "s_cmp_lt_i32 s0, s1", *filler(10), touch) == []


def test_accumulators_ahead_of_an_mfma():
    assert reasons("v_accvgpr_write_b32 a0, 0", *filler(2), MFMA) == ["an accumulation register is touched just ahead of an MFMA"]
    assert reasons("v_accvgpr_write_b32 a0, 0", *filler(3), MFMA) == []


@pytest.mark.parametrize("write", ["v_mov_b32_e32 v5, v30", "v_cndmask_b32_e32 v0, v1, v2, vcc", "v_lshl_add_u64 v[6:7], s[2:3], 0, v[30:31]"])
def test_operands_written_ahead_of_an_mfma(write):
    found = reasons(write, *filler(1), MFMA)
    assert found and all("just ahead of the MFMA that reads it" in x for x in found)
    assert reasons(write, *filler(2), MFMA) == []
    assert reasons("v_mov_b32_e32 v8, v30", MFMA) == []        # not an operand


@pytest.mark.parametrize("write", ["v_readlane_b32 s6, v40, 3", "v_readfirstlane_b32 s7, v2", "v_cmp_eq_u32_e64 s[6:7], v1, v2",
                                   "v_mad_u64_u32 v[1:2], s[6:7], v3, v4, 0"])
def test_scalar_base_of_a_direct_load(write):
    found = reasons(write, *filler(4), LOAD)
    assert found and all("the base of" in x for x in found)
    assert reasons(write, *filler(5), LOAD) == []
    assert reasons("s_add_u32 s6, s6, s0", LOAD) == []         # a scalar write needs no wait


def test_m0_ahead_of_a_direct_load():
    assert reasons("s_add_u32 m0, s4, 0x400", LOAD) == ["M0 is written just ahead of a direct load"]
    assert reasons("s_add_u32 m0, s4, 0x400", MFMA, LOAD) == []


# what a loop carries round: the copy stands far behind the last MFMA in the text, and right behind it on the way
LOOP = ["v_accvgpr_write_b32 a0, 0", "s_nop 15", ".LBB0_1:", "v_accvgpr_mov_b32 a9, a0", "s_nop 7", MFMA, "s_cmp_lt_i32 s0, s1"]


def test_back_edge():
    assert reasons(*LOOP, "s_cbranch_scc1 .LBB0_1") == ["an accumulation register is touched behind an MFMA"]
    assert reasons(*LOOP, "s_nop 9", "s_cbranch_scc1 .LBB0_1") == []
    assert reasons(*LOOP, "s_nop 7", "s_cbranch_scc1 .LBB0_1") == ["an accumulation register is touched behind an MFMA"]


def test_operand_written_at_the_bottom_of_a_loop():
    loop = [".LBB0_1:", MFMA, "s_nop 9", "v_mov_b32_e32 v1, v9"]
    assert reasons(*loop, "s_cbranch_vccnz .LBB0_1") == ["v1 is written by a vector instruction just ahead of the MFMA that reads it"]
    assert reasons(*loop, "s_nop 0", "s_cbranch_vccnz .LBB0_1") == []


def test_join_takes_the_shorter_way():
    body = [MFMA, "s_cbranch_scc1 .LBB0_2", "s_nop 15", ".LBB0_2:", "s_nop 9", "v_accvgpr_read_b32 v20, a0"]
    assert reasons(*body) == ["an accumulation register is touched behind an MFMA"]
    body[4] = "s_nop 10"
    assert reasons(*body) == []
    # code behind an unconditional branch is reached by its label only
    assert reasons(MFMA, "s_branch .LBB0_3", ".LBB0_2:", "v_accvgpr_read_b32 v20, a0", ".LBB0_3:", "s_nop 0") == []
