"""The generator of the assembly tiles refuses a schedule that reads a result too early."""
import importlib.util
import os

import pytest

PATH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_00023_amd", "csrc", "gen_fast_run.py")
spec = importlib.util.spec_from_file_location("gen_fast_run", PATH)
gen = importlib.util.module_from_spec(spec)
spec.loader.exec_module(gen)

MFMA = "v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], 0"
OTHER = "v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], 0"


@pytest.mark.parametrize("early,enough", [
    ([MFMA, "s_nop 6", "v_add_f32 v20, v2, v21"], [MFMA, "s_nop 7", "v_add_f32 v20, v2, v21"]),
    ([MFMA, OTHER, "s_nop 2", "v_add_f32 v20, v2, v21"], [MFMA, OTHER, "s_nop 3", "v_add_f32 v20, v2, v21"]),  # (the second waits for the pipe)
    (["v_exp_f32 v1, v2", "v_add_f32 v20, v1, v21"], ["v_exp_f32 v1, v2", "s_nop 0", "v_add_f32 v20, v1, v21"]),
    (["s_add_u32 m0, s59, 1024", "global_load_lds_dwordx4 v2, s[46:47]"], ["s_add_u32 m0, s59, 1024", "s_nop 0", "global_load_lds_dwordx4 v2, s[46:47]"]),
    (["v_xor_b32 v1, v2, v3", "s_nop 0", "v_xor_b32_dpp v4, v1, v5 row_newbcast:0 row_mask:0xf bank_mask:0xf"],
     ["v_xor_b32 v1, v2, v3", "s_nop 1", "v_xor_b32_dpp v4, v1, v5 row_newbcast:0 row_mask:0xf bank_mask:0xf"]),
    (["v_cmp_gt_i32 s[72:73], v1, 3", "s_nop 0", "v_cndmask_b32 v1, v2, v3, s[72:73]"],
     ["v_cmp_gt_i32 s[72:73], v1, 3", "s_nop 1", "v_cndmask_b32 v1, v2, v3, s[72:73]"]),
], ids=["matrix", "two matrix", "exponential", "m0", "broadcast", "comparison"])
def test_a_schedule_that_reads_too_early_is_refused(early, enough):
    gen.check_waits("tile", enough)
    with pytest.raises(AssertionError):
        gen.check_waits("tile", early)
