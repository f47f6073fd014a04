"""The build-time check of the distance between a vector write of a scalar register and a memory instruction that
reads it (csrc/check_sgpr_waits.py): planted early reads are reported, kept distances are not."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WRITE = "v_readfirstlane_b32 s3, v15"
STORE = "global_store_dwordx4 v6, a[0:3], s[2:3] sc1"


def _problems(body):
    path = os.path.join(ROOT, "paper_2603_05503_amd", "csrc", "check_sgpr_waits.py")
    spec = importlib.util.spec_from_file_location("check_sgpr_waits", path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    text = "\t.type\tkernel,@function\nkernel:\n"
    text += "".join(line + "\n" if line.endswith(":") else f"\t{line}\n" for line in body)
    return mod.check(text + ".Lfunc_end0:\n")


@pytest.mark.parametrize("body", [
    [WRITE, STORE, "s_endpgm"],
    [WRITE, "s_nop 3", STORE, "s_endpgm"],
    ["v_readlane_b32 s7, v1, 3", "s_mov_b32 m0, s9", "s_nop 0", "buffer_load_dwordx4 v1, s[4:7], s20 offen lds", "s_endpgm"],
    ["v_cmp_lt_i32_e64 s[20:21], v1, v2", "buffer_load_dword v1, v2, s[4:7], s20 offen", "s_endpgm"],
    [WRITE, "s_cbranch_scc1 .LBB0_2", "s_nop 7", STORE, "s_endpgm", ".LBB0_2:", "s_nop 0", STORE, "s_endpgm"],
])
def test_early_reads_are_reported(body):
    assert len(_problems(body)) == 1


@pytest.mark.parametrize("body", [
    [WRITE, "s_nop 4", STORE, "s_endpgm"],
    [WRITE, "s_mov_b32 s3, s5", STORE, "s_endpgm"],               # written again by the scalar unit
    [WRITE, "global_store_dwordx4 v3, a[0:3], s[4:5]", "s_endpgm"],  # another register
    ["s_mov_b32 s3, s5", STORE, "s_endpgm"],
    [WRITE, "v_add_f32 v1, v2, v3", "s_nop 1", "s_branch .LBB0_1", ".LBB0_1:", "s_nop 0", STORE, "s_endpgm"],
])
def test_kept_distances_pass(body):
    assert _problems(body) == []
