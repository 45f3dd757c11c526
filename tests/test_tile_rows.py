"""Tiles are found by prefixes of the tile schedule, which holds those of 64 and of 128 rows: other tile rows do not compile."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.parametrize("rows, ok", [(64, True), (128, True), (192, False), (256, False)])
def test_rows_of_a_token_tile(tmp_path, rows, ok):
    src = tmp_path / "rows.hip"
    src.write_text(f'#include "{ROOT}/paper_2406_04984_amd/csrc/gemm_mfma.h"\n'
                   f"__global__ void k(meft::TokenSched s, int* o) {{ meft::TileFinder f; f.init<{rows}>(s, 0, 1, false); o[0] = f.c; }}\n")
    p = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-device-only", "-fsyntax-only", str(src)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert (p.returncode == 0) == ok and ok == ("64 and of 128 rows" not in p.stdout), p.stdout[-3000:]
