"""fp32 key scores on the matrix cores at the edges of their tiles, against the oracle: groups around 32 and 64 rows, blocks
around multiples of 64 neurons, hidden sizes of less than one k tile (32), of one and of an odd and an even number with a
remainder, and enough tiles for the 64-row form."""
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=520, d=8, n_blocks=16, block_size=63, top_e=2, top_k=11),
    dict(T=700, d=32, n_blocks=20, block_size=65, top_e=1, top_k=9),
    dict(T=530, d=72, n_blocks=33, block_size=64, top_e=2, top_k=16, zipf_s=1.0),
    dict(T=640, d=104, n_blocks=10, block_size=130, top_e=1, top_k=30),
    dict(T=4203, d=40, n_blocks=4, block_size=1001, top_e=1, top_k=12),     # 64-row tiles
    dict(T=4203, d=136, n_blocks=4, block_size=960, top_e=1, top_k=12),
]


@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_d{k['d']}_{k['n_blocks']}x{k['block_size']}")
def test_against_the_oracle(kw):
    from tests import parity as P
    P.run_and_compare(synth.small_case(seed=8400 + kw["d"], dtype="f32", **kw)).assert_ok()
