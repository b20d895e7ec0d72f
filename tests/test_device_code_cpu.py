"""The device code as built: no packed-FP32 arithmetic, and the wait states that the compiler does not see to around inline
assembly.  The rules themselves on short pieces of assembly, then the library's own."""
import os

import pytest

from paper_2312_00752_amd import build, isa_check

# (instructions, findings)
PIECES = {
    "swap behind its operand's write": (["v_add_f32_dpp v1, v2, v2 row_ror:8 row_mask:0xf bank_mask:0xc", "s_nop 0",
                                         "v_permlane32_swap_b32_e32 v0, v1"], 1),
    "swap, first operand": (["v_mov_b32_e32 v0, v2", "v_permlane16_swap_b32_e32 v0, v1"], 1),
    "swap two wait states behind": (["v_mov_b32_e32 v0, v2", "s_nop 1", "v_permlane16_swap_b32_e32 v0, v1"], 0),
    "swap of a swap's result": (["v_permlane32_swap_b32 v0, v1", "v_mov_b32_e32 v5, v6", "v_permlane16_swap_b32 v1, v2"], 1),
    "swap behind other writes": (["v_mov_b32_e32 v3, v2", "v_permlane16_swap_b32_e32 v0, v1"], 0),
    "permuted operand": (["v_mul_f32_e32 v4, v2, v2", "s_waitcnt vmcnt(0)", "v_add_f32_dpp v1, v4, v3 quad_perm:[1,0,3,2] row_mask:0xf"], 1),
    "the operand that is not permuted": (["v_mul_f32_e32 v3, v2, v2", "v_add_f32_dpp v1, v4, v3 quad_perm:[1,0,3,2] row_mask:0xf"], 0),
    "matrix operand in a range": (["v_mov_b32_e32 v7, v2", "s_nop 0", "v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], 0"], 1),
    "transcendental": (["v_exp_f32_e32 v1, v2", "v_mul_f32_e32 v3, v1, v2"], 1),
    "transcendental, one apart": (["v_exp_f32_e32 v1, v2", "s_nop 0", "v_mul_f32_e32 v3, v1, v2"], 0),
    "accumulated onto": (["v_exp_f32_e32 v1, v2", "v_fmac_f32_e32 v1, v3, v2"], 1),
    "lane read": (["v_mov_b32_e32 v1, v2", "v_readfirstlane_b32 s0, v1"], 1),
    "across a label": (["v_mov_b32_e32 v0, v2", ".LBB0_1:", "v_permlane16_swap_b32_e32 v0, v1"], 1),
    "around a loop": (["s_nop 3", ".LBB0_1:", "v_permlane16_swap_b32_e32 v0, v1", "v_mov_b32_e32 v5, v1", "v_mov_b32_e32 v0, v2",
                       "s_cbranch_scc1 .LBB0_1"], 1),
    "past a jump": (["v_mov_b32_e32 v0, v2", "s_branch .LBB0_2", ".LBB0_1:", "v_permlane16_swap_b32_e32 v0, v1", ".LBB0_2:", "s_endpgm"], 0),
    "packed arithmetic": (["v_pk_add_f32 v[0:1], v[2:3], v[4:5]"], 1),
}


@pytest.mark.parametrize("name", sorted(PIECES))
def test_rules(name):
    lines, findings = PIECES[name]
    text = "kernel:\n" + "".join(("%s\n" if x.endswith(":") else "\t%s  ; a comment\n") % x for x in lines)
    found = isa_check.check(text)
    assert len(found) == findings, found


def test_library():
    if not build.device_assembly():
        build.build_library()
    files = build.device_assembly()
    assert len(files) == len(build.sources())
    for path in files:
        with open(path) as f:
            found = isa_check.check(f.read())
        assert not found, (os.path.basename(path), len(found), found[:3])
