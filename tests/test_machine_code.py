"""The library's GPU code as built: no instruction that subtracts with a DPP rotation in its reversed form.
The compiler makes one of x - rot(y), and the GPU computes rot(x) - y for it; the code is written so that
none is formed (pm_ptrans.h, pt_butterfly)."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2307_06554_amd as pm

LLVM = "/opt/rocm/llvm/bin"
REVERSED = re.compile(r"\bv_\w*rev_\w*_dpp\b")


def test_the_pattern():
    for line in ("v_subrev_u32_dpp v1, v2, v1 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1",
                 "v_subrev_co_u32_dpp v1, vcc, v2, v1 row_ror:3", "v_subbrev_co_u32_dpp v1, vcc, v2, v1, vcc row_ror:3"):
        assert REVERSED.search(line)
    for line in ("v_sub_u32_dpp v1, v1, v2 row_ror:3", "v_add_u32_dpp v1, v2, v1 row_ror:3", "v_subrev_u32_e32 v1, v2, v1"):
        assert not REVERSED.search(line)


@pytest.mark.skipif(not os.path.exists(LLVM + "/llvm-objdump") or shutil.which("objcopy") is None,
                    reason="no disassembler")
def test_no_reversed_subtraction_with_dpp(tmp_path):
    fat, code = str(tmp_path / "fat.bin"), str(tmp_path / "code.o")
    subprocess.run(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", pm.lib_path(), fat], check=True)
    subprocess.run([LLVM + "/clang-offload-bundler", "--type=o", "--unbundle", "--input=" + fat, "--output=" + code,
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    text = subprocess.run([LLVM + "/llvm-objdump", "-d", code], check=True, capture_output=True, text=True).stdout
    assert "v_sub_u32_dpp" in text  # the transform's own form: the code is there
    assert not sorted(set(REVERSED.findall(text)))
