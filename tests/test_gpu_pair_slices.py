"""The per-pair backward over column slices, against the oracle: rows of less than a slice (1 KB), of a few, of more than the
partial sums of ds have room for (8), a ragged last slice, segments of one pair, of more than a chunk (256) and of more than a
workgroup sorts in LDS (8192), fp32 and bf16."""
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(dtype="f32", T=37, d=8, n_blocks=4, block_size=40, top_e=2, top_k=9),
    dict(dtype="f32", T=600, d=264, n_blocks=3, block_size=17, top_e=2, top_k=20),          # a second slice of 8 columns
    dict(dtype="f32", T=90, d=2056, n_blocks=6, block_size=64, top_e=3, top_k=33),          # 9 slices: 8 groups, one of two
    dict(dtype="f32", T=40, d=16384, n_blocks=2, block_size=96, top_e=1, top_k=7),          # 64 slices
    dict(dtype="bf16", T=70, d=4104, n_blocks=4, block_size=80, top_e=2, top_k=21),         # 9 slices
    dict(dtype="bf16", T=520, d=1000, n_blocks=8, block_size=48, top_e=2, top_k=11, zipf_s=1.5),
    dict(dtype="bf16", T=33, d=512, n_blocks=1, block_size=70000, top_e=1, top_k=3),        # segments of one pair, 2^16 neurons
    dict(dtype="f32", T=9001, d=16, n_blocks=1, block_size=3, top_e=1, top_k=2),            # segments around 6000 pairs
    dict(dtype="f32", T=17000, d=8, n_blocks=1, block_size=2, top_e=1, top_k=2),            # 17000: ranked against LDS tiles
]


@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"{k['dtype']}_T{k['T']}_d{k['d']}_{k['n_blocks']}x{k['block_size']}")
def test_against_the_oracle(kw):
    from tests import parity as P
    P.run_and_compare(synth.small_case(seed=8300 + kw["T"], **kw)).assert_ok()
