"""The one-launch dispatch at its edges and just beyond its limits (where the chunked one takes over), against the oracle: tokens
around a workgroup's 1024, one and many blocks, as many entries and entries x blocks as it takes, groups of all sizes from none
to most of the batch, with the forward's tables reused by the backward and rebuilt (where a token may use fewer blocks)."""
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=1023, n_blocks=3, top_e=3, top_k=3), dict(T=1024, n_blocks=65, top_e=2, top_k=2), dict(T=1025, n_blocks=7, top_e=1, top_k=2),
    dict(T=2049, n_blocks=1024, top_e=4, top_k=4), dict(T=2048, n_blocks=1024, top_e=4, top_k=4, zipf_s=1.2),
    dict(T=16384, n_blocks=128, top_e=4, top_k=4), dict(T=16384, n_blocks=129, top_e=4, top_k=4),
    dict(T=16385, n_blocks=12, top_e=2, top_k=2, zipf_s=2.0), dict(T=9362, n_blocks=9, top_e=7, top_k=7), dict(T=9363, n_blocks=9, top_e=7, top_k=7),
    # chunked: 146 tokens per chunk, more than 512 blocks, more chunk counts than every workgroup adds up
    dict(T=16400, n_blocks=9, top_e=7, top_k=7), dict(T=3700, n_blocks=600, top_e=4, top_k=8), dict(T=9000, n_blocks=500, top_e=9, top_k=9),
]


@pytest.mark.parametrize("reuse", [False, True], ids=["rebuilt", "reused"])
@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_{k['n_blocks']}_e{k['top_e']}")
def test_against_the_oracle(kw, reuse):
    from tests import parity as P
    P.run_and_compare(synth.small_case(seed=8500 + kw["T"], dtype="bf16", d=64, block_size=16, reuse_fwd=reuse, **kw)).assert_ok()
