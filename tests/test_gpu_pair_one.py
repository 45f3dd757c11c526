"""The pairs of the per-pair backward grouped in one launch, against the oracle: one pair, fewer neurons than workgroups (128),
ragged ones, around the pairs (8192) and neurons (16384) up to which the kernel has its short form and buckets of more than four
neurons begin, segments that are sorted in LDS (more than 256 pairs) beside short ones, and all pairs in one segment."""
import numpy as np
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [  # T, n_blocks, block_size, top_e, top_k, dtype
    (1, 2, 8, 1, 1, "f32"), (700, 3, 37, 2, 5, "bf16"), (1031, 9, 113, 3, 7, "f32"), (8192, 1, 1, 1, 1, "f32"),
    (256, 64, 256, 1, 32, "f32"), (8193, 3, 40, 1, 1, "f32"), (500, 1, 16385, 1, 3, "bf16"), (4096, 2, 3, 1, 2, "f32"),
]


@pytest.mark.parametrize("T, nb, bs, e, k, dtype", CASES, ids=lambda v: str(v))
def test_against_the_oracle(T, nb, bs, e, k, dtype):
    from tests import parity as P
    P.run_and_compare(synth.small_case(seed=8800 + T, T=T, d=24, n_blocks=nb, block_size=bs, top_e=e, top_k=k, dtype=dtype)).assert_ok()


def test_long_and_short_segments():
    from tests.test_gpu_skew import _check, _hot_neurons
    t = _hot_neurons(synth.small_case(T=2000, d=16, n_blocks=1, block_size=600, top_e=1, top_k=4, dtype="f32", seed=8850),
                     {3: 10.0, 131: 9.0, 400: 0.3}, 7)
    n = np.bincount(_check(t)["idx"].ravel(), minlength=600)
    assert (n > 256).sum() >= 2 and ((n > 0) & (n <= 256)).sum() > 100
