"""Tiles looked up out of registers by the 128 x 256 and 256 x 256 contractions, against the oracle: more groups per XCD than one
load of a group list holds (63 or 64), fewer groups than XCDs (every list holds every group), and gathered token rows, through
buffer and through global loads."""
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=2100, d=128, n_blocks=1000, block_size=64, top_e=4, top_k=24),                # 125 groups per XCD, all small or nearly
    dict(T=3000, d=64, n_blocks=520, block_size=32, top_e=6, top_k=40, zipf_s=1.0),      # 65
    dict(T=1100, d=320, n_blocks=5, block_size=264, top_e=2, top_k=70, zipf_s=1.0),      # split lists, ragged tiles both ways
    dict(T=700, d=256, n_blocks=1, block_size=2048, top_e=1, top_k=20),                  # scores alone on the matrix cores
]


@pytest.mark.parametrize("forced", [False, True], ids=["buffer", "global"])
@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_d{k['d']}_{k['n_blocks']}x{k['block_size']}")
def test_against_the_oracle(kw, forced):
    from tests import parity as P
    from paper_2406_04984_amd import binding as B
    B.meft_debug_global_loads(forced)
    try:
        P.run_and_compare(synth.small_case(seed=8200 + kw["T"], dtype="bf16", **kw)).assert_ok()
    finally:
        B.meft_debug_global_loads(False)
