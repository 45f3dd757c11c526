"""The per-pair backward of few pairs, against the oracle: pairs grouped by buckets of one and of many neurons, up to what one launch
groups and one more; chunks of 1, 2, up to 4, up to 8, up to 64 and more pairs, several chunks of a neuron; rows of one to four and
more slices of 1 KB (1, 2 and 4 waves of a workgroup), ragged last slices; dV and dK out of one kernel and of two; tokens of fewer
pairs than a wave asks for rows together."""
import numpy as np
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

ONE_KERNEL = [  # T, d, n_blocks, block_size, top_e, top_k, dtype
    (3, 8, 2, 9000, 1, 5, "f32"), (40, 256, 1, 20000, 1, 30, "f32"), (70, 264, 3, 15, 2, 20, "f32"), (33, 776, 1, 4097, 1, 9, "f32"),
    (90, 1016, 6, 64, 3, 33, "f32"), (40, 2056, 1, 9000, 1, 30, "f32"), (8192, 16, 5, 1000, 1, 1, "f32"), (2731, 16, 5, 1000, 1, 3, "f32"),   # 8192, 8193 pairs
    (20480, 8, 2, 3000, 1, 1, "f32"), (20481, 8, 2, 3000, 1, 1, "f32"), (20481, 264, 1, 500, 1, 1, "f32"),
    (120, 512, 1, 4200, 1, 60, "bf16"), (120, 520, 1, 70000, 1, 60, "bf16"), (100, 1544, 1, 2600, 1, 4, "bf16"),
    (130, 40, 1, 7, 1, 2, "f32"), (260, 24, 1, 33, 1, 1, "f32"), (400, 72, 2, 11, 1, 4, "bf16"), (150, 24, 1, 33, 1, 9, "f32"),
]
TWO_KERNELS = [
    (90, 1032, 6, 64, 3, 33, "f32"),
    (700, 2056, 1, 900, 1, 12, "f32"), (300, 1000, 1, 30000, 1, 40, "f32"), (900, 4104, 1, 9000, 1, 11, "bf16"), (410, 784, 1, 5000, 1, 50, "f32"),
    (20480, 776, 1, 30000, 1, 1, "f32"), (20481, 776, 1, 30000, 1, 1, "f32"), (20481, 520, 1, 500, 1, 1, "f32"),
]


@pytest.mark.parametrize("T, d, nb, bs, e, k, dtype", ONE_KERNEL + TWO_KERNELS, ids=lambda v: str(v))
def test_against_the_oracle(T, d, nb, bs, e, k, dtype):
    from tests import parity as P
    P.run_and_compare(synth.small_case(seed=9100 + T + d, T=T, d=d, n_blocks=nb, block_size=bs, top_e=e, top_k=k, dtype=dtype)).assert_ok()


@pytest.mark.parametrize("T, d, N, k", [(2000, 16, 30000, 8), (2000, 784, 30000, 8), (5000, 16, 5000, 4), (700, 264, 100000, 20)])
def test_buckets_of_many_pairs(T, d, N, k):
    """Neighbouring neurons of one bucket that most tokens select: buckets of more pairs than a thread counts ranks among."""
    from tests.test_gpu_skew import _check, _hot_neurons
    base = N // 3 // 64 * 64
    hot = {base: 9.0, base + 1: 7.0, base + 2: 0.4, base + 3: 8.0, 17: 6.0, N - 1: 5.0}
    t = _hot_neurons(synth.small_case(T=T, d=d, n_blocks=1, block_size=N, top_e=1, top_k=k, dtype="f32", seed=9300 + T), hot, 7)
    n = np.bincount(_check(t)["idx"].ravel(), minlength=N)
    assert (n > 256).sum() >= 3 and ((n > 0) & (n <= 256)).sum() > 50
