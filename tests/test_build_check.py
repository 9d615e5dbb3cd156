"""The check that the build makes of the assembly of the inline-MFMA tile
kernels, on short listings of the form that the compiler writes."""
import pytest

from paper_2607_28144_amd.build import check_tile_kernels

NAME = "_ZN1k14linear4_kernelINS_6Shape4ILi8ELi8ELi3ELi1EEELi0EEEvi"
MFMA = "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\n"
WAITS = "\ts_nop 15\n\ts_nop 15\n"
READ = "\tv_accvgpr_read_b32 v0, a0\n"
ZERO = "\tv_accvgpr_write_b32 a0, 0\n"


def listing(body, name=NAME, spill=0, scratch=0):
    return (f"\t.text\n{name}: ; @{name}\n; %bb.0:\n{body}\ts_endpgm\n.Lfunc_end0:\n\t.size {name}, 1\n"
            f"amdhsa.kernels:\n  - .agpr_count: 4\n    .args:\n      - .offset: 0\n        .size: 4\n    .name:           {name}\n"
            f"    .private_segment_fixed_size: {scratch}\n    .sgpr_spill_count: 0\n    .symbol: {name}.kd\n"
            f"    .vgpr_spill_count: {spill}\n")


def loop(inside="", after=WAITS, before="\ts_nop 3\n", other=""):
    return (ZERO + before + ".LBB0_1: ; loop\n" + MFMA + inside + MFMA + "\ts_cbranch_scc1 .LBB0_1\n" +
            ("\ts_branch .LBB0_3\n.LBB0_2:\n" + other + ".LBB0_3:\n" if other else "") + after + READ)


def test_a_sound_kernel_passes():
    assert check_tile_kernels("t", listing(loop())) == 1
    # a block between the loop and its exit that no path from the loop enters
    assert check_tile_kernels("t", listing(loop(other=ZERO))) == 1


@pytest.mark.parametrize("body", [
    loop(inside="\tv_accvgpr_mov_b32 a4, a0\n"),        # a move between the MFMAs
    loop(after=""), loop(after="\ts_nop 15\n"),         # read with too few wait states
    loop(before=""), loop(before="\ts_nop 0\n"),        # written just before
    loop(after="\ts_cbranch_scc0 .LBB0_9\n" + WAITS + ".LBB0_9:\n"),  # a path around the wait states
])
def test_accumulators_touched_too_near(body):
    with pytest.raises(RuntimeError, match="accumulator"):
        check_tile_kernels("t", listing(body))


def test_spills_and_missing_resources():
    for text in (listing(loop(), spill=1), listing(loop(), scratch=8), listing(loop()).split("amdhsa.kernels")[0]):
        with pytest.raises(RuntimeError, match="spills"):
            check_tile_kernels("t", text)


def test_nothing_to_check_is_an_error():
    for text in ("", listing("\ts_nop 0\n"), listing(loop(), name=NAME.replace("Shape4", "Shape5"))):
        with pytest.raises(RuntimeError, match="no tile kernel"):
            check_tile_kernels("t", text)
