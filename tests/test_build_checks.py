"""The build's reading of the device assembly: an MFMA that the source writes out must not follow the write of one of its
operands by less than two wait states, on any path into it."""
import pytest

from paper_2501_16103_amd import build

MFMA = "v_mfma_f32_16x16x32_bf16 v[50:53], v[130:133], v[174:177], v[50:53]"
BY_HAND = f"\t;;#ASMSTART\n\t{MFMA}\n\t;;#ASMEND\n"


def _kernel(body):
    return f"_ZN3moe11gemm_kernelEv:                  ; @kernel\n; %bb.0:\n{body}\ts_endpgm\n.Lfunc_end0:\n"


REFUSED = {
    "accumulator_zeroed_before_the_loop": "\tv_mov_b32_e32 v53, v114\n\ts_add_i32 s4, s4, -2\n.LBB0_1:\n" + BY_HAND,
    "directly_behind": "\tv_mov_b32_e32 v50, 0\n" + BY_HAND,
    "fragment": "\tv_mov_b64_e32 v[174:175], v[2:3]\n\ts_nop 0\n" + BY_HAND,
    "second_path": "\ts_cbranch_scc1 .LBB0_2\n\ts_nop 3\n.LBB0_1:\n" + BY_HAND + "\ts_endpgm\n.LBB0_2:\n\tv_add_u32_e32 v130, 1, v2\n\ts_branch .LBB0_1\n",
    "back_edge": ".LBB0_1:\n" + BY_HAND + "\tv_mov_b32_e32 v52, 0\n\ts_cbranch_scc0 .LBB0_1\n",
}
ACCEPTED = {
    "two_wait_states": "\tv_mov_b32_e32 v53, v114\n\t;;#ASMSTART\n\ts_nop 1\n\t;;#ASMEND\n.LBB0_1:\n" + BY_HAND,
    "two_instructions": "\tv_mov_b32_e32 v53, v114\n\ts_add_i32 s4, s4, -2\n\ts_mov_b32 s5, 0\n" + BY_HAND,
    "other_registers": "\tv_mov_b32_e32 v54, v114\n" + BY_HAND,
    "read_only": "\tglobal_store_dword v[2:3], v53, off\n" + BY_HAND,
    "not_on_the_path": "\ts_nop 1\n\ts_branch .LBB0_1\n\tv_mov_b32_e32 v53, 0\n\ts_endpgm\n.LBB0_1:\n" + BY_HAND,
    "the_compilers_own": "\tv_mov_b32_e32 v53, v114\n\t" + MFMA + "\n",
}


@pytest.mark.parametrize("case", REFUSED)
def test_mfma_too_close_is_refused(case):
    with pytest.raises(RuntimeError, match="wait states behind"):
        build.check_mfma_operand_distance(_kernel(REFUSED[case]))


@pytest.mark.parametrize("case", ACCEPTED)
def test_mfma_far_enough_is_accepted(case):
    build.check_mfma_operand_distance(_kernel(ACCEPTED[case]))
