"""The build's check of where the compiler puts vector spills (text only, no compiler, no GPU)."""
from paper_1512_01383_amd.build import misplaced_spills

_KERNEL = """
_Z1kv:                                  ; @_Z1kv
; %bb.0:
	s_and_saveexec_b64 s[2:3], vcc
	s_cbranch_execz .LBB0_2
; %bb.1:
	v_add_u32_e32 v7, v1, v2
	scratch_store_dword off, v7, off offset:4 ; 4-byte Folded Spill
.LBB0_2:
	v_writelane_b32 v126, s8, 3
#	s_or_b64 exec, exec, s[2:3]
	scratch_store_dword off, v9, off offset:8 ; 4-byte Folded Spill
	s_endpgm
.Lfunc_end0:
"""
_SPILL = "\tscratch_store_dwordx2 off, v[90:91], off offset:32 ; 8-byte Folded Spill\n"
_RELOAD = "\tscratch_load_dword v5, off, off offset:16 ; 4-byte Folded Reload\n"
_USE = "\tglobal_store_dword v[2:3], v5, off\n"


def _kernel(lines):
    return _KERNEL.replace("#", lines)


def test_spills_ahead_of_the_other_lanes_return_are_found():
    assert misplaced_spills(_kernel("")) == []
    assert [k for k, _ in misplaced_spills(_kernel(_SPILL))] == ["_Z1kv"]
    assert misplaced_spills(_kernel("\tv_mov_b32_e32 v90, v1\n" + _SPILL)) == []   # the region's own
    assert [k for k, _ in misplaced_spills(_kernel(_RELOAD))] == ["_Z1kv"]
    assert misplaced_spills(_kernel(_RELOAD + _USE)) == []
