"""The check that the build runs over its own listing (build.py, dpp_hazards): DPP operands of inline asm need two wait states behind the
vector instruction that writes them (host code, no GPU)."""
import pytest

from paper_2509_05576_amd.build import dpp_hazards

USE = "\tv_fmac_f64_dpp v[24:25], -v[22:23], v[2:3] row_newbcast:1 row_mask:0xf bank_mask:0xf"


@pytest.mark.parametrize("lines", [
    ["\tv_mul_f64 v[22:23], v[4:5], v[6:7]", USE],                                             # written right before
    ["\tv_mul_f64 v[22:23], v[4:5], v[6:7]", "\ts_waitcnt lgkmcnt(0)", USE],                   # one wait state
    ["\tv_mov_b32_e32 v23, v4", "\ts_nop 0", USE],                                             # half of the pair
    ["\tv_accvgpr_read_b32 v22, a7", "\t;;#ASMSTART", USE],                                    # a spilled copy, a comment between
    ["\tv_permlane16_swap_b32 v9, v22", USE],                                                  # the second operand of a swap
    ["\tv_mul_f64 v[22:23], v[4:5], v[6:7]", "\ts_nop 1", USE.replace("v[24:25], -v[22:23]", "v[30:31], v[24:25]"),
     USE.replace("v[24:25], -v[22:23]", "v[32:33], v[30:31]")],                                # by the DPP instruction before
    ["\tv_mul_f64 v[22:23], v[4:5], v[6:7]", ".LBB0_3:", USE],                                 # behind a label: not known
    ["\tv_cmpx_gt_f64_e32 v[4:5], v[6:7]", "\ts_nop 3", USE],                                  # EXEC wants five
])
def test_hazards_are_found(lines):
    assert len(dpp_hazards("\n".join(lines))) == 1


@pytest.mark.parametrize("lines", [
    ["\tv_mul_f64 v[22:23], v[4:5], v[6:7]", "\ts_nop 1", USE],
    ["\tv_mul_f64 v[22:23], v[4:5], v[6:7]", "\tds_read_b64 v[22:23], v9", "\ts_waitcnt lgkmcnt(0)", USE],
    ["\tv_mul_f64 v[2:3], v[4:5], v[6:7]", USE],                                               # not the DPP operand
    ["\tv_mul_f64 v[24:25], v[4:5], v[6:7]", USE],
    ["\tv_mov_b32_e32 v21, v4", USE],
    [".LBB0_3:", "\ts_nop 1", USE],
    ["\tv_cmpx_gt_f64_e32 v[4:5], v[6:7]", "\ts_nop 4", USE],
    [USE, USE.replace("v[24:25]", "v[26:27]")],
])
def test_what_has_waited_long_enough_passes(lines):
    lines = ["\ts_nop 7"] + lines if not lines[0].startswith(".") else lines
    assert dpp_hazards("\n".join(lines)) == []
