"""The division by which a workgroup of the small-tile contraction finds its tile (csrc/tile_div.h), on the host: numbers of
m tiles around 65536, from where floor(w * ceil(2^32 / m) / 2^32) alone is one too large for some dividends, and the ends
of the range of its arguments."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_quotients_are_exact(tmp_path):
    exe = str(tmp_path / "tile_div_driver")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-fsanitize=undefined",
                           "-fno-sanitize-recover=all", "-o", exe, os.path.join(ROOT, "tests", "tile_div_driver.cpp")])
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert p.returncode == 0, p.stdout
