"""The build looks through the device listings for vector moves that a wavefront without active lanes would lose.  Small
listings, written by hand, with the move on either side of the restore."""
import pytest

from paper_2603_09221_amd import build

BODY = """
a_kernel:                               ; @a_kernel
; %%bb.0:
	v_cmp_gt_u32_e32 vcc, 64, v0
	s_and_saveexec_b64 s[4:5], vcc
	s_cbranch_execz .LBB0_2
; %%bb.1:
	v_add_f32_e32 v1, v1, v2
.LBB0_2:                                ; %%if.end
	%s
	v_readlane_b32 s6, v40, 3
	%s
	s_or_b64 exec, exec, s[4:5]
	%s
	v_mul_f32_e32 v1, v1, v3
	s_endpgm
"""
NOTHING = "s_nop 0"


@pytest.mark.parametrize("move", ["scratch_store_dword off, v7, off offset:128 ; 4-byte Folded Spill",
                                  "scratch_load_dwordx2 v[6:7], off, off offset:4", "v_accvgpr_write_b32 a3, v7",
                                  "v_mov_b32_e32 v9, v7"])
def test_a_move_ahead_of_the_restore_is_found(move):
    for text in (BODY % (move, NOTHING, NOTHING), BODY % (NOTHING, move, NOTHING)):
        assert [(k, x) for k, _, x in build.misplaced_vector_moves(text)] == [("a_kernel", move)]
    assert not build.misplaced_vector_moves(BODY % (NOTHING, NOTHING, move))


def test_joins_that_nobody_skips_to_and_other_code_are_left_alone():
    move = "scratch_store_dword off, v7, off offset:128"
    assert not build.misplaced_vector_moves((BODY % (move, NOTHING, NOTHING)).replace("s_cbranch_execz", "s_cbranch_scc0"))
    assert not build.misplaced_vector_moves(BODY % (move, "v_add_f32_e32 v4, v4, v4", NOTHING))
    assert not build.misplaced_vector_moves(BODY % (move, "s_and_b64 exec, exec, s[8:9]", NOTHING))


def test_flat_accesses_are_found():
    text = BODY % (NOTHING, "flat_load_dwordx4 v[0:3], v[4:5]", "flat_store_dword v[4:5], v0 offset:16")
    assert [(k, x.split()[0]) for k, _, x in build.flat_accesses(text)] == [("a_kernel", "flat_load_dwordx4"),
                                                                          ("a_kernel", "flat_store_dword")]
    assert not build.flat_accesses(BODY % (NOTHING, "global_load_dwordx4 v[0:3], v[4:5], off", "ds_read_b128 v[0:3], v4"))
    assert not build.flat_accesses("\t.amdhsa_uses_flat_scratch 0\n\t.max_flat_workgroup_size: 64\n; flat_load_dword v0, v[2:3]\n")


def test_spilled_registers_are_counted():
    """The kernels' metadata as the compiler writes it, the names of arguments before the kernel's own; every unit with a limit is built."""
    kernel = """  - .args:
      - .name:           p
        .size:           8
    .name:           %s
    .vgpr_count:     256
    .vgpr_spill_count: %d
"""
    text = "amdhsa.kernels:\n" + kernel % ("_ZN3ttc8a_kernelEv", 104) + kernel % ("_ZN3ttc8b_kernelEv", 0)
    assert build.spilled_registers(text) == [("_ZN3ttc8a_kernelEv", 104), ("_ZN3ttc8b_kernelEv", 0)]
    units = {(src, d) for src, sizes in build.UNITS for d in (sizes or (None,))}
    assert set(build.MOST_SPILLED) <= units
