"""The kernels' split asynchronous loads (load in one inline-assembly statement,
wait in a later one) as the compiler has laid them out: no instruction may
touch a destination register between the load and its wait.  CPU only: the
sources are compiled to assembly and scanned."""
import shutil

import pytest

from paper_2402_10876_amd import check_async_asm as chk

BAD = """
_Z1kv:
	;;#ASMSTART
	ds_read_b32 v35, v35
	;;#ASMEND
	v_mov_b32_e32 v76, v35
	;;#ASMSTART
	s_waitcnt lgkmcnt(0)
	;;#ASMEND
	s_endpgm
"""
GOOD = """
_Z1kv:
	;;#ASMSTART
	ds_read_b64_tr_b16 v[2:3], v9 offset:0
	;;#ASMEND
	;;#ASMSTART
	s_load_dwordx4 s[16:19], s[16:17], 0x0
	;;#ASMEND
	v_mfma_f32_32x32x16_f16 a[0:15], v[4:7], v[10:13], a[0:15]
	;;#ASMSTART
	s_waitcnt lgkmcnt(0)
	;;#ASMEND
	v_mov_b32_e32 v76, v2
	v_mov_b32_e32 v77, s17
	ds_read_b32 v1, v76
	v_mov_b32_e32 v5, v1
	s_endpgm
"""


# a single stage skips the wait of the loop: its accumulators may take the register of a row on its way
BAD_SKIP = """
_Z1kv:
	;;#ASMSTART
	global_load_dword v136, v134, s[4:5]
	;;#ASMEND
	s_cmp_lt_u32 s14, 2
	s_cbranch_scc1 .LBB0_2
	;;#ASMSTART
	s_waitcnt vmcnt(8)
	;;#ASMEND
	;;#ASMSTART
	v_mov_b32_dpp v119, v136 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf
	;;#ASMEND
	s_branch .LBB0_3
.LBB0_2:
	v_mov_b32_e32 v136, 0
.LBB0_3:
	;;#ASMSTART
	s_waitcnt vmcnt(0)
	;;#ASMEND
	s_endpgm
"""


# a spilled address comes back through v_readlane, and the load in the assembly block reads it five wait states too early
BAD_SPILL = """
_Z1kv:
	v_readlane_b32 s14, v105, 12
	v_readlane_b32 s15, v105, 13
	;;#ASMSTART
	global_load_dword v35, v92, s[14:15]
	;;#ASMEND
	;;#ASMSTART
	s_waitcnt vmcnt(0)
	;;#ASMEND
	s_endpgm
"""


def test_scanner_flags_a_scalar_address_that_a_vector_instruction_just_wrote():
    f = chk.check_scalar_addresses(BAD_SPILL)
    assert len(f) == 1 and f[0][0] == "_Z1kv" and f[0][3] == [("s", 14), ("s", 15)]
    load = "\tglobal_load_dword v35"
    assert len(chk.check_scalar_addresses(BAD_SPILL.replace(load, "\ts_nop 3\n" + load))) == 1
    assert chk.check_scalar_addresses(BAD_SPILL.replace(load, "\ts_nop 4\n" + load)) == []
    assert chk.check_scalar_addresses(BAD_SPILL.replace("v_readlane_b32 s1", "s_mov_b32 s1")) == []
    # the compiler's own instructions are its own business; a carry goes to the second operand, a mask to the first
    assert chk.check_scalar_addresses(BAD_SPILL.replace("\t;;#ASMSTART\n" + load, load)) == []
    for write in ("v_cmp_gt_i32_e64 s[14:15], v1, v2", "v_mad_u64_u32 v[2:3], s[14:15], v1, v2, v[4:5]"):
        assert len(chk.check_scalar_addresses(BAD_SPILL.replace("v_readlane_b32 s15, v105, 13", write))) == 1


def test_scanner_follows_the_vector_loads_along_branches():
    f = chk.check_branches(BAD_SKIP)
    assert len(f) == 1 and f[0][0] == "_Z1kv" and "v136, 0" in f[0][2]
    assert chk.check_branches(BAD_SKIP.replace("v_mov_b32_e32 v136", "v_mov_b32_e32 v137")) == []


def test_scanner_flags_a_use_before_the_wait_and_nothing_else():
    f = chk.check_assembly(BAD)
    assert len(f) == 1 and f[0][0] == "_Z1kv" and "v76, v35" in f[0][2]
    assert chk.check_assembly(GOOD) == []      # compiler-issued reads outside the markers are its own business


@pytest.mark.skipif(shutil.which(chk.HIPCC) is None, reason="hipcc not available")
def test_kernels_have_no_use_before_wait():
    assert chk.check_sources() == []
