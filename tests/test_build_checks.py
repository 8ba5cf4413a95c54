"""The build's check of products written as assembly, on listings with and without a hazard."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
spec = importlib.util.spec_from_file_location("glowq_build", os.path.join(ROOT, "paper_2603_25385_amd", "csrc", "build.py"))
hip_build = importlib.util.module_from_spec(spec)
spec.loader.exec_module(hip_build)

PRODUCT = "v_mfma_f32_16x16x32_f16 a[0:3], v[4:7], v[8:11], a[0:3]"


def check(*lines, kernel="k_wide"):
    text = "_Z6k_wide:\n" + "".join(l + "\n" if l.endswith(":") else f"\t{l}\n" for l in lines) + "\ts_endpgm\n"
    return hip_build.check_products("x.hip", text, kernel)


@pytest.mark.parametrize("lines", [
    ("v_mov_b32_e32 v4, v1", "s_nop 1", PRODUCT),
    ("v_mov_b32_e32 v12, v4", PRODUCT, "v_mov_b32_e32 v13, v4"),            # reads an operand, writes another register
    ("ds_read_b128 v[4:7], v1", "s_waitcnt lgkmcnt(0)", PRODUCT),           # a load's result is waited for
    (PRODUCT, PRODUCT, "s_nop 15", "s_nop 15", "v_accvgpr_read_b32 v1, a2"),
    ("v_mov_b32_e32 v4, v1", "s_branch .L2", ".L1:", PRODUCT, ".L2:", "s_nop 0"),
])
def test_listings_without_a_hazard(lines):
    assert check(*lines) >= 1


@pytest.mark.parametrize("lines", [
    ("v_mov_b32_e32 v7, v1", "s_nop 0", PRODUCT),                           # one state between
    ("v_permlane16_swap_b32_e32 v1, v9", PRODUCT),                          # its second register
    ("v_accvgpr_write_b32 a3, v1", PRODUCT),                                # the sum
    (PRODUCT, "s_nop 15", "v_accvgpr_read_b32 v1, a2"),                     # too early
    (PRODUCT, "s_nop 7", "global_store_dwordx4 v[1:2], a[0:3], off"),
    (".L1:", PRODUCT, "v_mov_b32_e32 v8, v1", "s_cbranch_scc0 .L1"),        # along the loop's back edge
    ("v_mfma_f32_16x16x32_f16 a[0:3], v[4:7], v[8:11], a[4:7]",),           # not in place
])
def test_hazards_are_found(lines):
    with pytest.raises(RuntimeError):
        check(*lines)


def test_other_kernels_are_left_to_the_compiler():
    assert check("v_mov_b32_e32 v7, v1", PRODUCT, kernel="k_other") == 0


NAMED = "v_mfma_scale_f32_16x16x128_f8f6f4 a[64:0x43], v[4:7], v[8:15], a[64:0x43], v1, v2 op_sel_hi:[0,0,0] cbsz:4"


@pytest.mark.parametrize("lines,ok", [
    (("v_accvgpr_write_b32 a[0x43], 0", "s_nop 1", NAMED, "s_nop 15", "s_nop 15", "v_accvgpr_read_b32 v1, a[0x42]"), True),
    ((NAMED, "s_nop 15", "v_accvgpr_read_b32 v1, a[0x42]"), False),                # too early
    (("v_accvgpr_write_b32 a[0x43], 0", NAMED), False),
    (("v_mov_b32_e32 v2, v9", "s_nop 0", NAMED), False),                           # a block scale
    (("v_accvgpr_write_b32 a9, v1", "s_nop 15", "s_nop 15", NAMED), False),        # something else in a sum's register
    (("ds_read_b128 a[0:3], v1", "s_nop 15", "s_nop 15", NAMED), False),
])
def test_sums_that_are_named_by_number(lines, ok):
    def run():
        text = "_Z9k_mx_wide:\n" + "".join(f"\t{l}\n" for l in lines) + "\ts_endpgm\n"
        return hip_build.check_products("x.hip", text, "k_mx_wide")

    if ok:
        assert run() == 1
    else:
        with pytest.raises(RuntimeError):
            run()
