"""The build's look at the assembly of the kernels that name registers themselves (no GPU needed; hipcc cross-compiles)."""
import os

import pytest

from paper_2511_12934_amd import asmcheck, build

META = "\t.amdhsa_kernel k\n    .private_segment_fixed_size: {scratch}\n    .vgpr_spill_count: {spill}\n"
MFMA = "\t;;#ASMSTART\n\tv_mfma_f32_32x32x16_bf16 {d}, v[100:103], v[104:107], {d}\n\t;;#ASMEND\n"


def check(body, spill=0, scratch=0):
    asmcheck.check("k:\n" + body + "\ts_endpgm\n" + META.format(spill=spill, scratch=scratch), "unit")


def mfma(d):
    return MFMA.format(d=d)


def nops(n):
    return "\ts_nop 0\n" * n


def test_accepts_what_the_kernels_do():
    check(mfma("v[0:15]") + mfma("v[0:15]") + mfma("a[0:15]") + mfma("a[16:31]") + mfma("a[32:47]") + "\tv_add_f32_e32 v60, v0, v1\n" +
          "\t;;#ASMSTART\n\tv_accvgpr_read_b32 v61, a[0]\n\tv_max_f32 v61, 0, v61\n\t;;#ASMEND\n")
    check(mfma("v[0:15]") + "\ts_nop 11\n\tv_mov_b32_e32 v60, v15\n")
    check("\tv_mov_b32_e32 v107, v1\n" + nops(2) + mfma("v[0:15]"))


@pytest.mark.parametrize("kw", [dict(spill=1), dict(scratch=16)])
def test_refuses_spills(kw):
    with pytest.raises(RuntimeError, match="wanted 0"):
        check(mfma("v[0:15]"), **kw)


@pytest.mark.parametrize("line", ["v_accvgpr_write_b32 a7, v3", "v_accvgpr_read_b32 v3, a255", "ds_read_b128 a[4:7], v1", "global_load_dword a1, v[2:3], off",
                                  "v_accvgpr_mov_b32 a1, a2"])
def test_refuses_accumulation_registers_in_the_compilers_hands(line):
    with pytest.raises(RuntimeError, match="accumulation register"):
        check(nops(40) + "\t" + line + "\n" + nops(40) + mfma("v[0:15]"))


@pytest.mark.parametrize("touch", ["v_mov_b32_e32 v60, v15", "v_mov_b32_e32 v15, 0", "ds_write_b32 v60, v3", "global_store_dwordx4 v60, v[12:15], s[0:1]"])
@pytest.mark.parametrize("between", [nops(11), "\ts_nop 10\n", mfma("a[0:15]") + nops(3)])
def test_refuses_a_touch_of_a_fresh_product(touch, between):
    with pytest.raises(RuntimeError, match="fresh results"):
        check(mfma("v[0:15]") + between + "\t" + touch + "\n")
    check(mfma("v[0:15]") + between + nops(1) + "\t" + touch + "\n")


def test_refuses_operands_that_are_not_there_yet():
    with pytest.raises(RuntimeError, match="fresh results"):
        check(mfma("v[100:115]") + mfma("v[0:15]"))
    with pytest.raises(RuntimeError, match="right behind"):
        check("\tv_mov_b32_e32 v107, v1\n" + nops(1) + mfma("v[0:15]"))


def test_follows_branches_back():
    loop = ".LBB0_1:\n\tv_mov_b32_e32 v60, v7\n" + nops(14) + mfma("v[0:15]") + "{gap}\ts_cbranch_scc1 .LBB0_1\n"
    check(loop.format(gap=nops(11)))
    with pytest.raises(RuntimeError, match="fresh results"):
        check(loop.format(gap=nops(10)))


def test_every_unit_that_names_them_is_checked():
    named = {f for f in build.sources() if '#include "k_mlp_acc.h"' in open(os.path.join(build.CSRC, f)).read()}
    assert named == set(build.CHECKED)


def test_the_build_fails_on_such_a_unit(tmp_path, monkeypatch):
    """A unit whose asm leaves an accumulation register to the compiler does not become an object."""
    body = ('#include <hip/hip_runtime.h>\ntypedef __bf16 b8 __attribute__((ext_vector_type(8)));\n'
            'typedef float f16 __attribute__((ext_vector_type(16)));\n'
            '__global__ void k(float *p, b8 *q)\n{\n    b8 a = q[threadIdx.x];\n    f16 c = {};\n'
            '    asm volatile("v_mfma_f32_32x32x16_bf16 %%0, %%1, %%1, %%0" : "+v"(c) : "v"(a));\n'
            '    asm volatile("s_nop 15");\n    asm volatile("; takes %%0" ::"%s"(p[1]));\n    p[threadIdx.x] = c[0];\n}\n')
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "_newest_header", lambda: 0.0)
    monkeypatch.setattr(build, "CHECKED", ("unit.hip",))
    (tmp_path / "unit.hip").write_text(body % "a")
    with pytest.raises(RuntimeError, match="the compiler uses an accumulation register"):
        build._compile("unit.hip", True)
    assert os.listdir(tmp_path) == ["unit.hip"]
    (tmp_path / "unit.hip").write_text(body % "v")
    assert os.path.exists(build._compile("unit.hip", True))
