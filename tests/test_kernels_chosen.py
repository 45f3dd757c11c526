"""That the GPU tests of a kernel reach it: which kernels their shapes launch, from the calls that the library makes of the HIP
runtime (tests/hostcalls.py)."""
import pytest

from tests.hostcalls import record, shape
from tests.test_gpu_not_finite import PAIRS
from tests.test_gpu_pair_rows import ONE_KERNEL, TWO_KERNELS
from tests.test_gpu_select_bound import CASES
from tests.test_gpu_union_rows import GATHERED, SMALL
from tests.test_gpu_wide_tiles import ALONE, EDGES, GRADIENTS, MASKED, SCORES, SPLIT, VALUES, group_sizes


def _names(calls, flags=0, **kw):
    rows, = record([(shape(flags=flags, **kw), calls)])
    return [r["name"] for r in rows if r["what"] == "launch"]


def _has(names, kernel):
    return any(kernel in n for n in names)


def test_selection_of_few_out_of_many():
    kernels = ("few_out", "select_reg", "select_bound", "select_big")
    got = record([(shape(**kw), ["fwd"]) for _, kw in CASES])
    for (kernel, kw), rows in zip(CASES, got):
        names = [r["name"] for r in rows]
        assert [k for k in kernels if _has(names, k)] == [kernel], (kw, names)


@pytest.mark.parametrize("N, T, kernel", [(5000, 6, "few_out"), (5000, 8, "few_out"), (5000, 40, "select_bound"),
                                          (30001, 8, "select_bound"), (20000, 6, "select_bound")])
def test_equal_keys_and_scores_that_are_no_numbers(N, T, kernel):
    assert _has(_names(["fwd"], T=T, d=64, n_blocks=1, block_size=N, top_e=1, top_k=100, dtype="f32"), kernel)


@pytest.mark.parametrize("few, kw", [
    (True, dict(T=48, d=64, n_blocks=6, block_size=64, top_e=2, top_k=30)),      # equal scores
    (False, dict(T=300, d=64, n_blocks=6, block_size=64, top_e=2, top_k=30)),
    (True, dict(T=64, d=64, n_blocks=8, block_size=32, top_e=3, top_k=20)),      # ties
    (False, dict(T=200, d=64, n_blocks=8, block_size=32, top_e=3, top_k=20)),
    (True, dict(T=96, d=128, n_blocks=40, block_size=32, top_e=2, top_k=4)),     # small groups only
    (False, dict(T=300, d=128, n_blocks=200, block_size=32, top_e=2, top_k=4))])
def test_few_tokens_and_block_dense(few, kw):
    names = _names(["fwd"], dtype="bf16", **kw)
    assert _has(names, "few_out") == few and _has(names, "select_reg") != few
    reuse = _names(["bwd"], flags=8, dtype="bf16", **kw)
    assert _has(reuse, "act_rows") == few      # the few-token forward leaves nothing to reuse


def test_pairs_of_the_per_pair_backward():
    for kernels, cases in PAIRS.items():
        for T, d, N, k in cases:
            names = _names(["bwd"], T=T, d=d, n_blocks=1, block_size=N, top_e=1, top_k=k, dtype="f32")
            assert all(_has(names, kernel) for kernel in kernels), (T, d, N, k, names)
    for cases, kernel in ((ONE_KERNEL, "seg_rows"), (TWO_KERNELS, "seg_dv")):
        for T, d, nb, bs, e, k, dtype in cases:
            names = _names(["bwd"], T=T, d=d, n_blocks=nb, block_size=bs, top_e=e, top_k=k, dtype=dtype)
            assert _has(names, kernel) and _has(names, "pair_one") == (T * k <= 20480), (T, d, nb, bs, k, names)


def test_gathered_rows_on_tiles_of_256_rows_and_of_128():
    names = [n for T, d, N, _, k in GATHERED
             for n in _names(["union_fwd", "union_bwd"], T=T, d=d, n_blocks=1, block_size=N, top_e=1, top_k=k, dtype="bf16")]
    for policy in ("TokKCRowsILi2E", "TokKCRowsILi1E", "TokNCRows", "NeuTNRows"):
        assert all(any(_has([n], kernel) and _has([n], policy) for n in names) for kernel in ("gemm_wide_kernel", "gemm_mfma_kernel")), policy


@pytest.mark.parametrize("call", ["union_fwd", "union_bwd"])
def test_rows_of_the_batch_union(call):
    for cases, gathered in ((GATHERED, True), (SMALL, False)):
        for T, d, N, _, k in cases:
            names = _names([call], T=T, d=d, n_blocks=1, block_size=N, top_e=1, top_k=k, dtype="bf16")
            assert _has(names, "gather_rows") != gathered and _has(names, "NCRows") == gathered, (T, d, N, k, names)


def test_tiles_of_256_rows():
    for sizes, kw, wide in EDGES:
        names = _names(["fwd", "bwd"], T=sum(group_sizes(sizes, kw["n_blocks"])), top_e=1, dtype="bf16", **kw)
        got = {p for p in (SCORES, MASKED, VALUES, GRADIENTS, ALONE) for n in names if _has([n], "gemm_wide_kernel") and _has([n], p)}
        assert got == set(wide), (kw, names)
    for kw in SPLIT:
        names = [n for n in _names(["fwd", "bwd"], dtype="bf16", **kw) if _has([n], "gemm_wide_kernel")]
        assert kw["n_blocks"] < 8 and all(_has(names, p) for p in (SCORES, MASKED, VALUES)), (kw, names)


# Forms of a token-major contraction, where the rounds of tiles decide: (call, shape, policy, on tiles of 256 rows?)
TOKEN_TILES = [
    ("fwd", dict(T=2048, d=1024, n_blocks=64, block_size=512, top_e=4, top_k=128), "ProbTokKCILi3E", False),
    ("fwd", dict(T=2048, d=4096, n_blocks=64, block_size=1024, top_e=4, top_k=256), "ProbTokKCILi3E", True),
    ("fwd", dict(T=8192, d=4096, n_blocks=64, block_size=1024, top_e=4, top_k=256), "ProbTokNC", True),
    ("fwd", dict(T=4096, d=4096, n_blocks=256, block_size=1024, top_e=8, top_k=512), "ProbTokNC", True),
    ("fwd", dict(T=2928, d=2688, n_blocks=28, block_size=864, top_e=1, top_k=200), "ProbTokNC", False),
    ("fwd", dict(T=8008, d=1472, n_blocks=18, block_size=816, top_e=1, top_k=100), "ProbTokNC", False),
    ("fwd", dict(T=2501, d=4992, n_blocks=28, block_size=896, top_e=3, top_k=99), "ProbTokNC", False),
    ("fwd", dict(T=138, d=3264, n_blocks=1, block_size=9984, top_e=1, top_k=100), "ProbTokKCILi0E", False),
    ("fwd", dict(T=137, d=2560, n_blocks=1, block_size=34560, top_e=1, top_k=100), "ProbTokKCILi0E", True),
    ("union_fwd", dict(T=879, d=1344, n_blocks=1, block_size=10240, top_e=1, top_k=64), "ProbTokNCRows", False),
    ("union_fwd", dict(T=1023, d=2048, n_blocks=32, block_size=512, top_e=4, top_k=128), "ProbTokNCRows", True),
]


@pytest.mark.parametrize("call, kw, policy, wide", TOKEN_TILES, ids=lambda v: f"T{v['T']}_d{v['d']}" if isinstance(v, dict) else str(v))
def test_rows_of_a_token_major_tile(call, kw, policy, wide):
    names = [n for n in _names([call], dtype="bf16", **kw) if _has([n], policy)]
    assert len(names) == 1 and _has(names, "gemm_wide_kernel" if wide else "gemm_mfma_kernel"), names


# The same of the weight gradients: (shape, on tiles of 256 rows?)
GRADIENT_TILES = [
    (dict(T=8192, d=4096, n_blocks=64, block_size=1024, top_e=4, top_k=256), True),
    (dict(T=4096, d=4096, n_blocks=256, block_size=1024, top_e=8, top_k=512), True),
    (dict(T=2048, d=1024, n_blocks=64, block_size=256, top_e=4, top_k=128), True),
    (dict(T=448, d=640, n_blocks=236, block_size=192, top_e=6, top_k=194), True),         # 58 MB
    (dict(T=808, d=768, n_blocks=40, block_size=720, top_e=2, top_k=56), False),          # 44 MB
    (dict(T=305, d=640, n_blocks=72, block_size=144, top_e=5, top_k=34), False),          # one k tile
    (dict(T=3480, d=768, n_blocks=88, block_size=192, top_e=1, top_k=10), False),
    (dict(T=1400, d=768, n_blocks=4, block_size=1024, top_e=1, top_k=64), False),         # 48 tiles of 256 rows
    (dict(T=1536, d=4096, n_blocks=64, block_size=300, top_e=2, top_k=64), False),        # 512 rows for 300
]


@pytest.mark.parametrize("kw, wide", GRADIENT_TILES, ids=lambda v: f"T{v['T']}_d{v['d']}" if isinstance(v, dict) else str(v))
def test_rows_of_a_weight_gradient_tile(kw, wide):
    names = [n for n in _names(["bwd"], dtype="bf16", **kw) if _has([n], "ProbNeuTN")]
    assert len(names) == 2 and all(_has([n], "gemm_wide_kernel" if wide else "gemm_mfma_kernel") for n in names), names
