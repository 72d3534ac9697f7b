"""Registers of the shape-agnostic attention kernels as they were built: no form spills, and the resident forms of heads of up to 64 leave
room for two blocks of eight waves on a compute unit where their launch rule counts on it."""
import os
import re
import subprocess

import pytest

from paper_2511_12934_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """mangled name -> (vector registers, bytes of scratch memory)"""
    build.build()
    d = tmp_path_factory.mktemp("co")
    fat, co = str(d / "fat"), str(d / "co")
    subprocess.check_call([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", os.path.join(build.OBJ, "k_generic.o"), str(d / "copy.o")])
    subprocess.check_call([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                           f"--input={fat}", f"--output={co}"])
    notes = subprocess.check_output([f"{LLVM}/llvm-readelf", "--notes", co], text=True)
    out = {}
    for k in notes.split("- .agpr_count:")[1:]:
        field = lambda n: re.search(rf"\.{n}:\s+(\S+)", k).group(1)  # noqa: E731
        out[field("name")] = int(field("vgpr_count")), int(field("private_segment_fixed_size"))
    return out


def test_no_form_spills(kernels):
    found = {n: v for n, v in kernels.items() if "k_attn_gen" in n and "generic" not in n}
    assert len(found) == 48                      # two types, four head widths, W_q or not, three kinds of block
    assert all(scratch == 0 for _, scratch in found.values()), found


@pytest.mark.parametrize("form", ["IfLi4ELi8ELb0ELb1E", "ItLi4ELi8ELb0ELb1E", "ItLi4ELi8ELb1ELb1E"])
def test_two_resident_blocks_a_compute_unit(kernels, form):
    (vgprs, _), = [v for n, v in kernels.items() if "k_attn_gen" + form in n]
    assert vgprs <= 128, vgprs                   # 512 a lane of a SIMD, two waves of each block on it
