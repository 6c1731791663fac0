"""The checks build.py runs on the generated assembly of the unit score kernel, on planted text: compiler code must stay
off the accumulation registers the kernel reserves, no ALU write may stand within two issue slots of the matrix
instruction that reads it, and nothing may read an accumulation register before the wait for its load."""
import pytest

from paper_2410_01518_amd import build

GOOD = """
\tv_cvt_pk_bf16_f32 v85, v24, v25
\ts_nop 1
\t;;#ASMSTART
\tv_mfma_f32_32x32x16_bf16 v[34:49], v[82:85], a[0:3], 0
\t;;#ASMEND
\tv_add_f32_e32 v100, v2, v3
\tv_add_f32_e32 v104, v2, v3
\t;;#ASMSTART
\tv_mfma_f32_32x32x16_bf16 v[2:17], v[0:3], a[32:35], v[2:17]
\t;;#ASMEND
\t;;#ASMSTART
\tglobal_load_dwordx4 a[8:11], v[20:21], off offset:32
\t;;#ASMEND
"""


def _write(tmp_path, text):
    p = tmp_path / "k.s"
    p.write_text(text)
    return str(p)


def test_clean_text_passes(tmp_path):
    p = _write(tmp_path, GOOD)
    build.check_acc_registers_untouched(p)
    build.check_matrix_operand_distance(p)


@pytest.mark.parametrize("gap", ["", "\tv_mov_b32_e32 v200, v201\n"])
def test_alu_write_directly_before_the_matrix_instruction_that_reads_it_is_refused(tmp_path, gap):
    text = "\tv_cvt_pk_bf16_f32 v85, v24, v25\n" + gap + "\tv_mfma_f32_32x32x16_bf16 v[34:49], v[82:85], a[0:3], 0\n"
    with pytest.raises(RuntimeError, match="matrix instruction"):
        build.check_matrix_operand_distance(_write(tmp_path, text))


def test_two_slots_in_between_are_enough_and_the_accumulator_operand_does_not_count(tmp_path):
    ok = ("\tv_cvt_pk_bf16_f32 v85, v24, v25\n\tv_mov_b32_e32 v200, v201\n\tv_mov_b32_e32 v202, v201\n"
          "\tv_mfma_f32_32x32x16_bf16 v[34:49], v[82:85], a[0:3], 0\n"
          "\tv_add_f32_e32 v40, v1, v2\n\tv_mfma_f32_32x32x16_bf16 v[34:49], v[86:89], a[0:3], v[34:49]\n")
    build.check_matrix_operand_distance(_write(tmp_path, ok))


def test_compiler_code_on_an_accumulation_register_is_refused(tmp_path):
    with pytest.raises(RuntimeError, match="accumulation registers"):
        build.check_acc_registers_untouched(_write(tmp_path, GOOD + "\tv_accvgpr_write_b32 a5, v1\n"))
    with pytest.raises(RuntimeError, match="accumulation registers"):
        build.check_acc_registers_untouched(_write(tmp_path, GOOD + "\tv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]\n"))


LOAD, WAIT = "\tglobal_load_dwordx4 a[0:3], v[20:21], off\n", "\ts_waitcnt vmcnt(0)\n"
MMA = "\tv_mfma_f32_32x32x16_bf16 v[34:49], a[0:3], v[82:85], 0\n"


def test_matrix_instruction_behind_the_wait_is_accepted(tmp_path):
    build.check_acc_loads_awaited(_write(tmp_path, "kernel:\n" + LOAD + WAIT + MMA + "\ts_endpgm\n"))
    # the wait in a loop that loads again; what follows an s_branch is not reached from before it
    build.check_acc_loads_awaited(_write(tmp_path, "kernel:\n.LBB0_1:\n" + LOAD + WAIT + MMA + "\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n"))
    build.check_acc_loads_awaited(_write(tmp_path, "kernel:\n" + LOAD + "\ts_branch .LBB0_2\n.LBB0_1:\n" + MMA + ".LBB0_2:\n" + WAIT + MMA))


@pytest.mark.parametrize("text", [
    LOAD + "\ts_waitcnt vmcnt(1)\n" + MMA,                                                    # a wait that counts other loads
    LOAD + "\ts_cbranch_scc1 .LBB0_2\n" + WAIT + ".LBB0_2:\n" + MMA,                          # a way around the wait
    ".LBB0_1:\n" + MMA + LOAD + "\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n"])                   # from one round of a loop to the next
def test_matrix_instruction_that_a_load_may_reach_is_refused(tmp_path, text):
    with pytest.raises(RuntimeError, match="under way"):
        build.check_acc_loads_awaited(_write(tmp_path, "kernel:\n" + text))
