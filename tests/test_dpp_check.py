"""The build's check of the broadcast operands on written-out listings: what
reaches a broadcast too soon, on a straight path, over a branch and over a long
branch, and what does not."""
import pytest

from paper_2108_10565_amd import dpp_check

FMAC = "v_fmac_f64_dpp v[42:43], v[2:3], v[88:89] row_newbcast:0 row_mask:0xf bank_mask:0xf"
NOP = "s_mov_b32 s0, 0"


def _listing(lines):
    """objdump's form, four bytes per instruction; "-> k" marks a branch to line k."""
    out = ["0000000000001000 <kernel>:"]
    for i, line in enumerate(lines):
        text, _, to = line.partition(" -> ")
        note = f" <kernel+0x{4 * int(to):x}>" if to else ""
        out.append(f"\t{text:<58} // {0x1000 + 4 * i:012X}: 00000000{note}")
    return "\n".join(out)




@pytest.mark.parametrize("lines,bad", [
    (["ds_read_b64 v[2:3], v1", "s_waitcnt lgkmcnt(0)", FMAC], 0),             # as the kernel has it
    (["v_mov_b32_e32 v3, v9", FMAC], 1),                                       # a copy right before
    (["v_mov_b32_e32 v3, v9", NOP, FMAC], 1),                                  # one wait state
    (["v_mov_b32_e32 v3, v9", NOP, NOP, FMAC], 0),                             # two
    (["v_mov_b32_e32 v3, v9", "s_nop 1", FMAC], 0),
    (["v_accvgpr_read_b32 v2, a4", "s_nop 0", FMAC], 1),                       # a spill comes back
    (["v_mov_b32_e32 v88, v9", "v_mov_b32_e32 v4, v9", FMAC], 0),              # other operands and registers
    (["v_lshl_add_u64 v[2:3], v[8:9], 0, v[6:7]", FMAC], 1),                   # a pair
    (["v_swap_b32 v9, v3", FMAC], 1),                                          # writes both
    (["v_mov_b32_e32 v3, v9", "s_cbranch_scc1 1 -> 4", NOP, NOP, FMAC], 1),    # over the branch only
    (["v_mov_b32_e32 v3, v9", "s_branch 1 -> 3", NOP, FMAC], 1),
    (["s_branch 2 -> 3", "v_mov_b32_e32 v3, v9", "s_branch 1 -> 4", FMAC, "s_endpgm"], 0),  # not on its path
    (["v_cmpx_gt_u32_e32 5, v0", NOP, NOP, NOP, FMAC], 1),                     # EXEC
    (["v_cmpx_gt_u32_e32 5, v0", "s_nop 4", FMAC], 0),
])
def test_listings(lines, bad):
    count, found = dpp_check.hazards(_listing(lines))
    assert count == 1 and len(found) == bad, found


@pytest.mark.parametrize("copy_at,bad", [(None, 0), (3, 1)])
def test_long_branch(copy_at, bad):
    """s_getpc .. s_setpc back to a broadcast: distances count from the
    instruction after s_getpc; the compiler writes backward ones as 32 bits."""
    lines = [NOP, FMAC, "s_endpgm", "s_getpc_b64 s[0:1]", f"s_add_u32 s0, s0, 0x{(4 - 16) & 0xffffffff:x}",
             "s_addc_u32 s1, s1, -1", "s_setpc_b64 s[0:1]"]
    if copy_at is not None:  # a copy in the middle of the sequence would be too soon
        lines[5] = "v_mov_b32_e32 v2, v9"
    count, found = dpp_check.hazards(_listing(lines))
    assert count == 1 and len(found) == bad, found
