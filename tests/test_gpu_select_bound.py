"""Selection of few out of many candidates: both sides of the candidate counts and of the top_k that this kernel takes, key
counts per thread, counts that are no multiple of 4 or of its sweep, and more equal keys than its list holds (tokens of
zeros, keys that all repeat), where it falls back to exact passes and the lower ids have to win."""
import numpy as np
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

# with the kernel that selects: the bound one, the one that holds all keys in registers, the forward of few tokens or, beyond
# 65536 candidates, the one that goes through memory
CASES = [
    ("few_out", dict(T=20, d=64, n_blocks=1, block_size=4097, top_e=1, top_k=40, dtype="f32")),
    ("few_out", dict(T=32, d=64, n_blocks=1, block_size=8193, top_e=1, top_k=257, dtype="f32")),
    ("select_reg", dict(T=33, d=64, n_blocks=1, block_size=4096, top_e=1, top_k=40, dtype="f32")),
    ("select_bound", dict(T=33, d=64, n_blocks=1, block_size=4097, top_e=1, top_k=40, dtype="f32")),
    ("select_bound", dict(T=70, d=64, n_blocks=2, block_size=4100, top_e=2, top_k=256, dtype="f32")),
    ("select_bound", dict(T=40, d=64, n_blocks=1, block_size=8193, top_e=1, top_k=256, dtype="f32")),
    ("select_reg", dict(T=40, d=64, n_blocks=1, block_size=8193, top_e=1, top_k=257, dtype="f32")),
    ("select_bound", dict(T=40, d=128, n_blocks=1, block_size=12288, top_e=1, top_k=100, dtype="bf16")),
    ("select_bound", dict(T=150, d=128, n_blocks=1, block_size=12300, top_e=1, top_k=1, dtype="bf16")),
    ("select_bound", dict(T=20, d=64, n_blocks=3, block_size=9001, top_e=3, top_k=200, dtype="bf16")),
    ("select_bound", dict(T=10, d=64, n_blocks=1, block_size=65536, top_e=1, top_k=256, dtype="f32")),
    ("select_big", dict(T=10, d=64, n_blocks=1, block_size=65540, top_e=1, top_k=30, dtype="f32")),
]


@pytest.mark.parametrize("kernel, kw", CASES, ids=[f"{n}_T{k['T']}_C{k['top_e'] * k['block_size']}_k{k['top_k']}" for n, k in CASES])
def test_parity(kernel, kw):
    from tests import parity as P
    P.run_and_compare(synth.small_case(seed=8100 + kw["block_size"], **kw)).assert_ok()


@pytest.mark.parametrize("N, T", [(5000, 8), (5000, 40), (30001, 8)])
def test_more_equal_keys_than_the_list_holds(N, T):
    from tests import parity as P
    cfg = synth.small_case(T=T, d=64, n_blocks=1, block_size=N, top_e=1, top_k=100, dtype="f32", seed=8200)
    t = synth.make_inputs(cfg)
    t.h[:3] = 0.0                       # every score 0: the first 100 neurons
    t.K[:] = t.K[np.arange(N) % 2]      # two distinct keys: the better one's first 100 positions
    g = P.run_gpu(t)
    assert (g["idx"][:3] == np.arange(100)).all()
    s = t.h @ t.K[:2].T
    best = (s[3:, 1] > s[3:, 0]).astype(int)
    assert (g["idx"][3:] == best[:, None] + 2 * np.arange(100)[None]).all()


@pytest.mark.parametrize("N, T", [(5000, 6), (5000, 40), (20000, 6)])
def test_scores_that_are_no_numbers(N, T):
    from tests import parity as P
    k = 100
    t = synth.make_inputs(synth.small_case(T=T, d=64, n_blocks=1, block_size=N, top_e=1, top_k=k, dtype="f32", seed=8300))
    ref = P.run_gpu(t)["idx"]
    t.h[1] = np.nan            # every score of the token
    t.K[[7, 1999, 4321]] = np.nan   # three scores of every token: they rank above the numbers, or all of them below
    idx = P.run_gpu(t)["idx"]
    assert (idx >= 0).all() and (idx < N).all() and (np.diff(idx, axis=1) > 0).all()
    for i in range(T):
        if i == 1:
            continue
        rest = np.setdiff1d(idx[i], [7, 1999, 4321])
        assert len(rest) in (k, k - 3) and np.isin(rest, ref[i]).sum() >= k - 3
