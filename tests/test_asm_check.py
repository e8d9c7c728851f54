"""The check of the compiled assembly around asm statements, on texts with planted mistakes."""
import glob
import os

import pytest

from paper_2311_09431_amd import asm_check, build

MFMA = "v_mfma_f32_32x32x16_bf16 %s, %s, %s, %s"


def by_hand(*lines):
    return [";;#ASMSTART", *lines, ";;#ASMEND"]


def kernel(*lines, name="wide_kernel"):
    return "\n".join(["%s: ; @%s" % (name, name), *("\t" + x for x in lines), "\ts_endpgm", ".Lfunc_end0:"])


OWN = by_hand("s_nop 1", MFMA % ("a[0:15]", "v[0:3]", "v[4:7]", "a[0:15]"))
SCORE = by_hand(MFMA % ("v[16:31]", "v[0:3]", "v[4:7]", "0"))
OTHER = by_hand(MFMA % ("a[16:31]", "v[0:3]", "v[4:7]", "a[16:31]"))


@pytest.mark.parametrize("lines,found", [
    (OWN + ["v_add_f32_e32 v8, v9, v10"] + OWN, None),
    (OWN + ["v_accvgpr_write_b32 a200, v8"] + OWN, "a200"),
    (OWN + ["v_accvgpr_read_b32 v8, a15"] + OWN, "a15"),
    (OWN + [MFMA % ("a[240:255]", "v[0:3]", "v[4:7]", "a[240:255]")], "a[240:255]"),
    (OWN + ["s_mov_b32 s1, s2 ; a1 in a comment"], None),
    (["s_nop 0"], "no kernel"),
])
def test_accumulators_by_number(lines, found):
    findings = asm_check.check(kernel(*lines), ["wide_kernel"])
    assert (found is None) == (not findings) and all(found in x for x in findings), findings


def test_a_kernel_that_is_not_there():
    assert asm_check.check(kernel(*OWN, name="other"), ["wide_kernel"])


@pytest.mark.parametrize("lines,found", [
    # an operand just written: 0 and 1 wait states, 2, another register, by a memory read (which has its own wait)
    (["v_cvt_pk_bf16_f32 v3, v8, v9"] + OTHER, True),
    (["v_cvt_pk_bf16_f32 v3, v8, v9", "s_mov_b32 s0, 0"] + OTHER, True),
    (["v_cvt_pk_bf16_f32 v3, v8, v9", "s_mov_b32 s0, 0", "s_mov_b32 s1, 0"] + OTHER, False),
    (["v_cvt_pk_bf16_f32 v3, v8, v9", "s_nop 1"] + OTHER, False),
    (["v_cvt_pk_bf16_f32 v3, v8, v9"] + OWN, False),
    (["v_cvt_pk_bf16_f32 v8, v3, v9"] + OTHER, False),
    (["v_permlane32_swap_b32_e32 v8, v3"] + OTHER, True),
    # registers as asm statements print their constants
    (by_hand("v_accvgpr_write_b32 a[0xa1], v8", MFMA % ("v[16:31]", "v[0:3]", "a[0xa0:0xa3]", "0")), True),
    (by_hand("v_accvgpr_write_b32 a[63], v8", MFMA % ("v[16:31]", "v[0:3]", "a[60:63]", "0")), True),
    (by_hand("v_accvgpr_write_b32 a[0xa4], v8", MFMA % ("v[16:31]", "v[0:3]", "a[0xa0:0xa3]", "0")), False),
    (["ds_read_b128 v[0:3], v9", "s_waitcnt lgkmcnt(0)"] + OTHER, False),
    # around a loop and over a branch
    ([".LBB0_1:", "s_nop 0"] + OTHER + ["s_cbranch_scc1 .LBB0_2", "v_mov_b32_e32 v4, v9", "s_branch .LBB0_1", ".LBB0_2:"], False),
    ([".LBB0_1:"] + OTHER + ["s_cbranch_scc1 .LBB0_2", "v_mov_b32_e32 v4, v9", "s_branch .LBB0_1", ".LBB0_2:"], True),
    # a result that has not landed: read, overwritten, stored, a factor; after 10 and 11 wait states, after products
    (SCORE + ["v_exp_f32_e32 v8, v20"], True),
    (SCORE + ["v_mov_b32_e32 v31, 0"], True),
    (SCORE + ["ds_write_b32 v9, v16"], True),
    (SCORE + [MFMA % ("v[40:55]", "v[16:19]", "v[4:7]", "0")], True),
    (SCORE + ["s_nop 9", "v_exp_f32_e32 v8, v20"], True),
    (SCORE + ["s_nop 10", "v_exp_f32_e32 v8, v20"], False),
    (SCORE + OTHER + ["v_exp_f32_e32 v8, v20"], True),
    (SCORE + OTHER + OTHER + ["v_exp_f32_e32 v8, v20"], False),
    (SCORE + SCORE + ["v_exp_f32_e32 v8, v20"], True),
    (SCORE + ["v_exp_f32_e32 v8, v9"], False),
    (OWN + by_hand("v_accvgpr_read_b32 v8, a15"), True),
    (OWN + OWN + by_hand("s_nop 15", "v_accvgpr_read_b32 v8, a15"), False),
    # (the compiler sees to its own)
    ([MFMA % ("v[16:31]", "v[0:3]", "v[4:7]", "0"), "v_exp_f32_e32 v8, v20"], False),
])
def test_waits(lines, found):
    findings = asm_check.check(kernel(*lines))
    assert bool(findings) == found, findings


def test_the_build_ends_at_a_finding(tmp_path, monkeypatch):
    monkeypatch.setitem(build.ASM_CHECKED, "x.hip", ["wide_kernel"])
    obj, asm = tmp_path / "x.o", tmp_path / "x-hip-amdgcn-amd-amdhsa-gfx950.s"
    obj.write_text(""), asm.write_text(kernel(*OWN))
    build._check_asm("x.hip", str(obj))
    assert obj.exists() and not asm.exists()
    asm.write_text(kernel(*OWN, "v_mov_b32_e32 v8, a3"))
    with pytest.raises(RuntimeError, match="names an accumulator"):
        build._check_asm("x.hip", str(obj))
    assert not obj.exists()


def test_every_source_with_such_statements_is_checked():
    users = set()
    for path in glob.glob(os.path.join(build.CSRC, "*.hip")):
        with open(path) as f:
            text = f.read()
        if '"v_mfma' in text or "\\tv_mfma" in text or "mfma_vgpr_" in text:
            users.add(os.path.basename(path))
    assert users and users <= set(build.ASM_CHECKED)
