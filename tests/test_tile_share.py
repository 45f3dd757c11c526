"""The deal of tiles to the XCDs where there are fewer groups than XCDs (csrc/tile_share.h), on the host: every tile once, and as
many to each XCD, whether a group has one column of tiles or many."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_tile_once_in_even_parts(tmp_path):
    exe = str(tmp_path / "tile_share_driver")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-fsanitize=undefined,address",
                           "-fno-sanitize-recover=all", "-o", exe, os.path.join(ROOT, "tests", "tile_share_driver.cpp")])
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert p.returncode == 0, p.stdout
