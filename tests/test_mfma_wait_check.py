"""The build-time check of the distance behind an MFMA or a dot product (csrc/check_mfma_waits.py): planted early uses in a piece of
device assembly are reported on straight paths, behind branches and around loops; kept distances are not."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _problems(body):
    path = os.path.join(ROOT, "paper_2603_05503_amd", "csrc", "check_mfma_waits.py")
    spec = importlib.util.spec_from_file_location("check_mfma_waits", path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    text = "\t.type\tkernel,@function\nkernel:\n"
    text += "".join(line + "\n" if line.endswith(":") else f"\t{line}\n" for line in body)
    return mod.check(text + ".Lfunc_end0:\n")


MFMA = "v_mfma_f32_32x32x16_bf16 v[18:33], v[2:5], v[6:9], v[18:33]"
ACC = "v_mfma_f32_32x32x16_f16 a[0:15], v[2:5], v[6:9], 0"
READ = "v_mul_f32_e32 v3, s59, v18"
DOT = "v_dot2c_f32_bf16 v18, 0x3f803f80, v[0x5e]"


@pytest.mark.parametrize("body", [
    [MFMA, "s_nop 10", READ, "s_endpgm"],
    [MFMA, "s_nop 10", "v_mov_b32_e32 v33, 0", "s_endpgm"],                       # a write of the result
    [MFMA, "s_nop 3", "ds_write_b32 v1, v20", "s_endpgm"],
    [ACC, "s_nop 4", "v_accvgpr_read_b32 v2, a7", "s_endpgm"],
    [ACC, "s_nop 4", "global_store_dwordx4 v[0:1], a[12:15], off", "s_endpgm"],
    [MFMA, "v_mfma_f32_32x32x16_bf16 v[40:55], v[20:23], v[6:9], 0", "s_endpgm"],  # as an operand
    [MFMA, "v_mfma_f32_32x32x16_bf16 v[34:49], v[2:5], v[6:9], v[18:33]", "s_endpgm"],  # moved, not chained
    [MFMA, "s_cbranch_scc1 .LBB0_2", "s_nop 15", READ, "s_endpgm", ".LBB0_2:", "s_nop 3", READ, "s_endpgm"],
    [MFMA, "s_branch .LBB0_2", ".LBB0_1:", READ, "s_endpgm", ".LBB0_2:", "s_nop 8", "s_branch .LBB0_1"],
    [".LBB0_1:", READ, "s_nop 15", MFMA, "s_nop 1", "s_cbranch_vccnz .LBB0_1", "s_endpgm"],  # around a loop
    ["v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], 0", "s_endpgm"],          # a shape without a known distance
    [DOT, "s_setprio 0", "s_andn2_b64 vcc, exec, s[2:3]", READ, "s_endpgm"],       # a dot product: three states
    [DOT, "v_mov_b32_e32 v18, 0", "s_endpgm"],
    [DOT, "v_dot2c_f32_bf16 v19, v18, v20", "s_endpgm"],                           # as an operand of another sum
    [DOT, "v_dot2c_f32_f16 v18, v1, v20", "s_endpgm"],                             # another kind of dot product
    [DOT, "s_cbranch_vccnz .LBB0_2", "s_nop 3", ".LBB0_2:", READ, "s_endpgm"],
])
def test_early_uses_are_reported(body):
    assert len(_problems(body)) == 1


@pytest.mark.parametrize("body", [
    [MFMA, "s_nop 11", READ, "s_endpgm"],
    [MFMA, MFMA, "s_nop 0xb", READ, "s_endpgm"],                                   # accumulation into the same registers
    [MFMA, "v_mfma_f32_32x32x16_bf16 v[18:33], v[2:5], v[6:9], 0", "s_nop 11", READ, "s_endpgm"],  # or a new sum in them
    [DOT, "s_nop 2", READ, "s_endpgm"],
    [DOT, DOT, "v_cvt_pk_bf16_f32 v[0x5f], v33, v34", "s_nop 1", READ, "s_endpgm"],  # the sum goes on
    [MFMA, "s_nop 9", "s_cbranch_scc1 .LBB0_2", "s_nop 0", ".LBB0_2:", "s_nop 0", READ, "s_endpgm"],
    [MFMA, "v_mul_f32_e32 v3, s59, v17", "v_mul_f32_e32 v34, s59, a18 ; v18", "s_endpgm"],
    [MFMA, "s_nop 3", "s_branch .LBB0_2", ".LBB0_1:", READ, "s_endpgm", ".LBB0_2:", "s_nop 7", "s_branch .LBB0_1"],
])
def test_kept_distances_pass(body):
    assert _problems(body) == []
