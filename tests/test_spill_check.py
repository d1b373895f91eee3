"""The build's look through its device assembly for vector-register spills stored
ahead of a block's restored execution mask."""
import pytest

from paper_2507_02888_amd.spill_check import misplaced_spills

KERNEL = "_ZN5ewald5k_runILi3EEEvPKNS_6DevSysE:\n"


def found(body):
    return misplaced_spills([KERNEL] + [x + "\n" for x in body.strip("\n").split("\n")])


@pytest.mark.parametrize("store", ["scratch_store_dwordx2 off, v[10:11], off offset:16 ; 8-byte Folded Spill",
                                   "v_accvgpr_write_b32 a3, v10 ;  Reload Reuse"])
def test_spill_at_a_loop_exit_is_found(store):
    got = found(f"""
.LBB0_7:                                ;   Parent Loop BB0_3 Depth=1
\tv_add_f64 v[0:1], v[0:1], v[2:3]
\ts_andn2_b64 exec, exec, s[4:5]
\ts_cbranch_execnz .LBB0_7
; %bb.8:                                ;   in Loop: Header=BB0_3 Depth=1
\tv_writelane_b32 v255, s30, 5
\ts_waitcnt vmcnt(0)
\t{store}
\ts_or_b64 exec, exec, s[6:7]
""")
    assert len(got) == 1 and got[0][0].startswith("_ZN5ewald5k_run") and got[0][1] == store.strip()


@pytest.mark.parametrize("body", [
    # after the mask is restored
    """
; %bb.8:
\ts_or_b64 exec, exec, s[6:7]
\tscratch_store_dword off, v1, off
""",
    # work of the narrower mask itself, stored before the lanes join
    """
.LBB0_9:
\tv_add_f64 v[0:1], v[0:1], v[2:3]
\tscratch_store_dwordx2 off, v[0:1], off
\ts_or_b64 exec, exec, s[6:7]
""",
    # no join in this block
    """
.LBB0_9:
\tscratch_store_dword off, v1, off
\ts_cbranch_scc1 .LBB0_12
; %bb.10:
\ts_or_b64 exec, exec, s[6:7]
""",
])
def test_other_spills_are_not(body):
    assert found(body) == []
