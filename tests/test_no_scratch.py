"""The contractions hold everything in registers and LDS: a function of theirs that the compiler does not inline puts policy, tile and
finder into scratch memory, which costs 5 to 10 % of their time and changes no result.  Read from the built library's kernel
descriptions."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2406_04984_amd", "libmeft.so")
LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-readelf")), reason="no ROCm LLVM tools")
def test_contractions_use_no_scratch_memory(tmp_path):
    fat, obj = str(tmp_path / "fat"), str(tmp_path / "gfx950.co")
    subprocess.check_call([os.path.join(LLVM, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", LIB, str(tmp_path / "copy")])
    subprocess.check_call([os.path.join(LLVM, "clang-offload-bundler"), "--unbundle", "--type=o", f"--input={fat}",
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--output={obj}"])
    notes = subprocess.check_output([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], text=True)
    kernels = dict(re.findall(r"\.name: +(\S+)\n.*?\.private_segment_fixed_size: +(\d+)", notes, re.S))
    gemms = {n: int(b) for n, b in kernels.items() if "gemm_wide" in n or "gemm_mfma" in n or "gemm_tile" in n}
    assert len(gemms) > 20 and not any(gemms.values()), {n: b for n, b in gemms.items() if b}
