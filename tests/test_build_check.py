"""The build's check of the GEMM kernels' machine code (build.py), on made-up
disassembly: what it refuses, in which sources."""
import pytest

from paper_2407_17353_amd import build

MID8 = "_ZN7scalify15mid_gemm_kernelILb0ELb0ELi0ELi%dELi8ELi3EEEvNS_10GemmParamsE"
MID4 = "_ZN7scalify15mid_gemm_kernelILb0ELb0ELi0ELi0ELi4ELi4EEEvNS_10GemmParamsE"
WAVE = "_ZN7scalify16wave_gemm_kernelILb0ELb0ELi0ELi0ELb0ELi4EEEvNS_10GemmParamsE"
MFMA = "v_mfma_f32_16x16x128_f8f6f4 a[0:3], v[0:7], v[8:15], a[0:3]"
SPILL = "scratch_store_dword off, v1, s32"


def mid(extra=()):
    return {**{MID8 % i: [MFMA, *extra] for i in range(4)}, MID4: [MFMA, "v_accvgpr_write_b32 a0, v3"]}


def test_sound_kernels_pass():
    assert build.check_functions("/x/mid_nn.hip.o", mid()) == 4
    assert build.check_functions("/x/gemm_nn.hip.o", {"k": [MFMA, "v_accvgpr_read_b32 v1, a0"]}) == 1
    assert build.check_functions("/x/gemm_nn_fused.hip.o", {"k": [SPILL]}) == 0
    assert build.check_functions("/x/wave_nn.hip.o", {WAVE: ["v_mfma_f32_16x16x128_f8f6f4 v[0:3], v[4:11], v[12:19], 0"]}) == 0


@pytest.mark.parametrize("obj,functions", [
    ("/x/wave_nn.hip.o", {WAVE: [SPILL]}),
    ("/x/mid_nn.hip.o", {**mid(), MID4: [MFMA, SPILL]}),
    ("/x/mid_nn.hip.o", mid([SPILL])),
    ("/x/gemm_nn.hip.o", {"k": [MFMA, SPILL]})], ids=["wave", "mid128", "mid256", "gemm"])
def test_scratch_memory_is_refused(obj, functions):
    with pytest.raises(RuntimeError, match="scratch"):
        build.check_functions(obj, functions)


def test_held_accumulators_are_left_alone():
    with pytest.raises(RuntimeError, match="AGPR"):
        build.check_functions("/x/mid_nn.hip.o", mid(["v_accvgpr_write_b32 a0, v3"]))
    with pytest.raises(RuntimeError, match="AGPR"):
        build.check_functions("/x/gemm_nn.hip.o", {"k": [MFMA], "f": ["v_accvgpr_write_b32 a0, v3"]})


def test_a_mid_kernel_of_another_form_does_not_go_unchecked():
    """Another template argument must not switch the check off."""
    with pytest.raises(RuntimeError, match="another form"):
        build.check_functions("/x/mid_nn.hip.o", {"_ZN7scalify15mid_gemm_kernelILb0ELi8ELi3EEEvv": [MFMA]})
    with pytest.raises(RuntimeError, match="not 4"):
        build.check_functions("/x/mid_nn.hip.o", {MID4: [MFMA]})


def test_scalar_operands_keep_their_distance():
    near = ["v_readlane_b32 s16, v2, 0", "s_mov_b32 m0, s3", "s_nop 0", "buffer_load_dword v2, s[16:19], 0 offen lds"]
    far = near[:2] + ["s_nop 3"] + near[3:]
    assert build.scalar_distance_violations(near) and not build.scalar_distance_violations(far)
