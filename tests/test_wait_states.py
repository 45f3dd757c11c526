"""A buffer load reads its descriptor and its offset from scalar registers.  Where a vector instruction has written one of them
(v_readlane of a spilled register, v_readfirstlane, a comparison), the hardware wants five wait states in between.  The compiler
sees to them, but not in front of an asm block, where gemm_wide_kernel has its loads: here every direct load of the built library is
looked at, back over the instructions before it."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2406_04984_amd", "libmeft.so")
LLVM = "/opt/rocm/llvm/bin"
STATES = 5


def _scalars(operand):
    """numbers of the scalar registers that an operand names"""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m[1])} if m else set()


def _too_early(code):
    """the loads of a kernel's instructions that come too early: (index, the instruction before)"""
    bad = []
    for i, line in enumerate(code):
        op, *args = re.split(r"[ ,]+", line)
        if not (op.startswith("buffer_load") and "lds" in args):
            continue
        reads = set().union(*map(_scalars, args))
        states, j = 0, i - 1
        while j >= 0 and states < STATES:
            before, *to = re.split(r"[ ,]+", code[j])
            if before.startswith("v_") and any(_scalars(t) & reads for t in to[:2 if "_co_" in before or "div_scale" in before else 1]):
                bad.append((i, code[j]))
            states += int(to[0], 0) + 1 if before == "s_nop" else 1
            j -= 1
    return bad


def test_the_check_itself():
    load = "buffer_load_dwordx4 v1, s[8:11], s4 offen lds"
    gap = ["s_add_i32 m0, s5, 0x400", "s_nop 0"]
    assert not _too_early(["v_readlane_b32 s9, v2, 3", "s_nop 2", *gap, load])
    assert _too_early(["v_readlane_b32 s9, v2, 3", "s_nop 1", *gap, load])
    assert _too_early(["v_readfirstlane_b32 s4, v2", *gap, load]) and not _too_early(["v_readfirstlane_b32 s5, v2", *gap, load])
    assert _too_early(["v_cmp_eq_u32_e64 s[10:11], v2, v3", *gap, load])


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objdump")), reason="no ROCm LLVM tools")
def test_direct_loads_of_the_library(tmp_path):
    fat, obj = str(tmp_path / "fat"), str(tmp_path / "gfx950.co")
    subprocess.check_call([os.path.join(LLVM, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", LIB, str(tmp_path / "copy")])
    subprocess.check_call([os.path.join(LLVM, "clang-offload-bundler"), "--unbundle", "--type=o", f"--input={fat}",
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--output={obj}"])
    text = subprocess.check_output([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", "--mcpu=gfx950", obj], text=True)
    loads = 0
    for kernel in re.split(r"\n(?=[0-9a-f]+ <)", text):
        if "gemm_wide_kernel" not in kernel.partition("\n")[0]:
            continue
        code = [l.split("//")[0].strip() for l in kernel.split("\n")[1:] if l.startswith("\t")]
        loads += sum(c.startswith("buffer_load") and c.endswith(" lds") for c in code)
        assert not _too_early(code), (kernel.partition("\n")[0], _too_early(code)[:3])
    assert loads > 200
