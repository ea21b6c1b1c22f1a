"""Registers of kernels whose time hangs on a second workgroup per CU, from the
metadata of the built objects: 512-lane workgroups need 128 VGPRs or fewer for it."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2109_14704_amd", "_build")
LLVM = "/opt/rocm/llvm/bin/"


def vgprs(obj, tmp_path):
    """{kernel symbol: VGPRs} of an object file's gfx950 code."""
    fat, co = str(tmp_path / "fat"), str(tmp_path / "co")
    subprocess.check_call([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj])
    subprocess.check_call([LLVM + "clang-offload-bundler", "--type=o", "--unbundle", "--input=" + fat, "--output=" + co,
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"])
    notes = subprocess.check_output([LLVM + "llvm-readelf", "--notes", co], text=True)
    return {re.search(r"\.name:\s+(\S+)", b).group(1): int(re.search(r"\.vgpr_count:\s+(\d+)", b).group(1))
            for b in notes.split("- .agpr_count")[1:]}


@pytest.mark.skipif(not os.path.exists(os.path.join(BUILD, "tr_prod_grouped.o")) or not os.path.exists(LLVM + "llvm-readelf"),
                    reason="needs the built objects and the LLVM tools")
@pytest.mark.parametrize("obj,kernel", [("tr_prod_tensor.o", "k_prod"), ("tr_prod_grouped.o", "k_prod_g")])
@pytest.mark.parametrize("log_n", [11, 12])
def test_tensor_of_ntt_inputs_keeps_two_workgroups(tmp_path, obj, kernel, log_n):
    name = "%sILi%dELi%dELi%dELi3ELi1ELb0ELb1EE" % (kernel, log_n, log_n, log_n)   # <N, ST, B, E = 3, tensor, no fwd, inv>
    got = [v for k, v in vgprs(os.path.join(BUILD, obj), tmp_path).items() if name in k]
    assert len(got) == 1 and got[0] <= 128, got
