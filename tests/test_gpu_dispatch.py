"""The grouping of the (token, block) entries at the edges of its chunks and of its limits: entries per token that do not
divide a chunk, one chunk and many, more blocks or chunk counts than every workgroup adds up for itself, groups around
the sizes that the deal to the XCDs treats apart (64 rows), a touched list of several chunks and one beyond the flags that
a workgroup counts itself; tables rebuilt by the backward and reused."""
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=600, d=64, n_blocks=9, block_size=64, top_e=7, top_k=70),                      # 146 tokens per chunk
    dict(T=513, d=64, n_blocks=8, block_size=16, top_e=2, top_k=8),                       # eight groups, one per XCD
    dict(T=700, d=64, n_blocks=7, block_size=16, top_e=2, top_k=8),                       # fewer groups than XCDs
    dict(T=450, d=128, n_blocks=70, block_size=32, top_e=10, top_k=40, zipf_s=1.0),       # groups of 1 .. 450 rows
    dict(T=2000, d=64, n_blocks=31, block_size=16, top_e=1, top_k=4),                     # groups around 64 rows
    dict(T=300, d=64, n_blocks=600, block_size=16, top_e=4, top_k=8),                     # more than 512 blocks
    dict(T=9000, d=64, n_blocks=500, block_size=16, top_e=9, top_k=12, zipf_s=0.8),       # 80 chunks x 500 blocks
    dict(T=2044, d=64, n_blocks=1024, block_size=16, top_e=513, top_k=130),               # 2044 chunks, just under 2^20 entries
    dict(T=300, d=64, n_blocks=1030, block_size=16, top_e=2, top_k=8),                    # the general path
    dict(T=1500, d=64, n_blocks=140, block_size=1000, top_e=2, top_k=64),                 # 140000 neurons
]


@pytest.mark.parametrize("reuse", [False, True])
@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_B{k['n_blocks']}x{k['block_size']}_e{k['top_e']}")
def test_parity(kw, reuse):
    from tests import parity as P
    cfg = synth.small_case(seed=5100 + kw["T"], dtype="bf16", reuse_fwd=reuse, **kw)
    P.run_and_compare(cfg).assert_ok()
