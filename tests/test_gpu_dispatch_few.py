"""The one-launch dispatch of many tokens to few blocks, against the oracle: where it begins (4097 tokens, 2 blocks) and ends (64
blocks, 16384 tokens, 3584 entries per block), every number of parts that a block's tokens are placed in, steps that are looked
through one at a time, popular blocks, tables of the forward reused and rebuilt (where a token may use fewer blocks)."""
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=4097, n_blocks=2, top_e=1, top_k=1), dict(T=7168, n_blocks=2, top_e=1, top_k=2, zipf_s=1.0),   # 32 parts for 5 and 7 steps
    dict(T=5000, n_blocks=11, top_e=3, top_k=2), dict(T=8192, n_blocks=14, top_e=6, top_k=6, zipf_s=1.5),  # 5 and 4 parts
    dict(T=16384, n_blocks=32, top_e=4, top_k=4, zipf_s=1.2), dict(T=16383, n_blocks=22, top_e=4, top_k=3),  # 2 parts
    dict(T=12289, n_blocks=32, top_e=2, top_k=2), dict(T=16384, n_blocks=64, top_e=4, top_k=4, zipf_s=1.2),                     # 1
]


@pytest.mark.parametrize("reuse", [False, True], ids=["rebuilt", "reused"])
@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_{k['n_blocks']}_e{k['top_e']}")
def test_against_the_oracle(kw, reuse):
    from tests import parity as P
    P.run_and_compare(synth.small_case(seed=8900 + kw["T"], dtype="bf16", d=64, block_size=16, reuse_fwd=reuse, **kw)).assert_ok()
