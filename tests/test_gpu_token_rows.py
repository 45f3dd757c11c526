"""Sums of a token's partial rows against the oracle where they are read through L2 (60 to 190 MB of them, contractions of one k
tile): one and two 16-byte pieces of a row per thread, tokens in fewer blocks than they may be in, and groups that are summed pair
by pair beside them."""
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=1000, d=4096, n_blocks=16, block_size=64, top_e=8, top_k=64),
    dict(T=2100, d=2048, n_blocks=24, block_size=32, top_e=8, top_k=24, zipf_s=1.5),
]


@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_d{k['d']}")
def test_partial_rows_read_through_l2(kw):
    from tests import parity as P
    assert 60 << 20 <= kw["T"] * kw["top_e"] * kw["d"] * 2 <= 190 << 20 and kw["block_size"] <= 192
    P.run_and_compare(synth.small_case(seed=9100 + kw["T"], dtype="bf16", **kw)).assert_ok()
