"""Launch shapes of accepted problems against the limits of the device (65536 workgroups along y and z, fewer than 2^32
threads along x, 1024 threads and 160 KB of LDS per workgroup), at the far ends of what the shape check lets through and
a batch can hold."""
import pytest

from tests.hostcalls import record, shape

CASES = [
    (shape(3_000_000, 8, 8, 1, 1, 1, "f32"), ["route", "fwd", "bwd"]),
    (shape(10_000_000, 16, 1, 4, 1, 4, "f32"), ["route", "fwd", "bwd"]),
    (shape(3_000_000, 72, 2, 16, 2, 8, "bf16"), ["route", "fwd", "bwd"]),
    (shape(4_194_305, 64, 1, 64, 1, 1, "bf16"), ["route", "fwd", "bwd"]),
    (shape(400_000, 64, 64, 16, 8, 16, "bf16"), ["route", "fwd", "bwd"]),
    (shape(1, 16384, 16384, 1, 1, 1, "f32"), ["route", "fwd", "bwd"]),
    (shape(512, 16384, 512, 96, 1, 96, "bf16"), ["route", "fwd", "bwd"]),
    (shape(70_000, 128, 16384, 8, 3, 5, "f32"), ["route", "fwd", "bwd"]),
    (shape(500, 64, 1, 4_194_304, 1, 4096, "bf16"), ["route", "fwd", "bwd"]),
    (shape(100_000, 64, 4, 512, 2, 64, "bf16"), ["union_fwd", "union_bwd"]),
    (shape(20_000_000, 8, 8, 16, 1, 1, "f32"), ["bwd"]),
    (shape(16_384, 2056, 16_384, 860, 1, 860, "bf16"), ["route", "fwd", "bwd"]),
]


@pytest.fixture(scope="module")
def launches():
    return [[r for r in rows if r["what"] == "launch"] for rows in record(CASES)]


@pytest.mark.parametrize("i", range(len(CASES)), ids=lambda i: "T{}_d{}_N{}_B{}".format(*CASES[i][0][:4]))
def test_within_the_limits_of_the_device(launches, i):
    assert launches[i]
    for r in launches[i]:
        g, b = r["grid"], r["block"]
        assert min(g) >= 1 and g[1] <= 65536 and g[2] <= 65536, r
        assert g[0] * b[0] < 1 << 32 and b[0] * b[1] * b[2] <= 1024 and r["lds"] <= 160 * 1024, r


# The router contraction without LDS tiles re-reads its operands; beyond what the first shape of each pair has it took up
# to five times as long as the tiled ones (1404 against 274 us at 16384 x 4104 bf16 and 1024 blocks).
ROUTER = [
    (shape(4096, 4096, 8, 64, 4, 16, "bf16"), shape(8192, 4096, 8, 64, 4, 16, "bf16"), "gemm_mfma_kernel"),
    (shape(4096, 4096, 64, 64, 4, 16, "bf16"), shape(4097, 4096, 64, 64, 4, 16, "bf16"), "gemm_mfma_kernel"),
    (shape(2048, 5120, 32, 64, 4, 16, "bf16"), shape(5000, 5120, 32, 64, 4, 16, "bf16"), "gemm_mfma_kernel"),
    (shape(5000, 4224, 8, 64, 4, 16, "bf16"), shape(8192, 4224, 32, 64, 4, 16, "bf16"), "gemm_mfma_kernel"),
    (shape(8192, 4160, 8, 64, 4, 16, "bf16"), shape(20000, 4160, 8, 64, 4, 16, "bf16"), "gemm_mfma_kernel"),
    (shape(32768, 1024, 8, 64, 4, 16, "bf16"), shape(32768, 2048, 8, 64, 4, 16, "bf16"), "gemm_mfma_kernel"),
    (shape(12000, 2112, 3, 64, 3, 16, "bf16"), shape(16000, 2112, 3, 64, 3, 16, "bf16"), "gemm_mfma_kernel"),
    (shape(4096, 4104, 64, 64, 4, 16, "bf16"), shape(16384, 4104, 64, 64, 4, 16, "bf16"), "gemm_nt_"),
    (shape(16384, 1000, 64, 64, 4, 16, "bf16"), shape(16384, 1000, 1024, 64, 4, 16, "bf16"), "gemm_nt_"),
    (shape(16384, 1024, 64, 64, 4, 16, "f32"), shape(16384, 1024, 256, 64, 4, 16, "f32"), "gemm_nt_"),
    (shape(4096, 512, 64, 64, 4, 16, "f32"), shape(16384, 512, 1024, 64, 4, 16, "f32"), "gemm_nt_"),
]


def test_large_router_contractions_run_on_tiles():
    rows = record([(s, ["route"]) for untiled, tiled, _ in ROUTER for s in (untiled, tiled)])
    for (untiled, tiled, name), a, b in zip(ROUTER, rows[::2], rows[1::2]):
        assert "route_part_kernel" in a[0]["name"], (untiled, a)
        assert name in b[0]["name"], (tiled, b)


# The selection with sixteen keys per lane took 153 us where the one with keys in LDS takes 112 (16384 tokens, 1024 blocks,
# top_e 16), 92 against 40 with top_e 1.
@pytest.mark.parametrize("T, n_blocks, top_e, name", [
    (16384, 256, 1, "route_pick_kernel"), (2048, 1024, 8, "route_pick_kernel"), (2049, 1024, 8, "route_topk_kernel"),
    (2048, 257, 7, "route_topk_kernel"), (100, 1025, 8, "route_topk_kernel")])
def test_selection_of_blocks(T, n_blocks, top_e, name):
    rows, = record([(shape(T, 64, n_blocks, 64, top_e, 16, "bf16"), ["route"])])
    assert [name in r["name"] for r in rows] == [False, True], rows


# Chunks hold whole tokens (1023 entries of 1024 at top_e 3), and the limit is on the entries: counted in chunks, the last
# thousand below 2^20 entries fell to kernels that scan all entries once per block (2338 instead of 1560 us at 349400 x 3).
@pytest.mark.parametrize("T, n_blocks, top_e, chunked", [
    (349_525, 64, 3, True), (349_526, 64, 3, False), (1_048_576, 8, 1, True), (1_048_577, 8, 1, False),
    (2044, 1024, 513, True), (1_048_576 // 513 + 1, 1024, 513, False)])
def test_dispatch_in_chunks_up_to_its_limit(T, n_blocks, top_e, chunked):
    rows, = record([(shape(T, 64, n_blocks, 16, top_e, 8 * top_e, "bf16"), ["fwd"])])
    assert any("dispatch_place" in r["name"] for r in rows) == chunked, rows


def test_token_rows_keep_their_lists_short():
    # a list of all of top_k in LDS: 104 us for the rows that took 61 without (4096 tokens x 8 entries x 4096, top_k 8192)
    rows, = record([(shape(4096, 4096, 16, 1024, 8, 8192, "bf16"), ["fwd", "bwd"])])
    rows = [r for r in rows if "token_rows" in r["name"]]
    assert len(rows) == 2 and all(r["lds"] <= 8192 for r in rows), rows


# Gradient rows of small groups in the launch of the dh rows leave most of its waves idle where rows are short and many.
@pytest.mark.parametrize("T, d, own", [(300_000, 64, True), (32_768, 512, True), (8192, 1024, False), (8193, 1024, True),
                                       (8192, 4096, False), (2048, 512, False)])
def test_gradient_rows_of_small_groups_share_a_launch(T, d, own):
    rows, = record([(shape(T, d, 64, 16, 2, 8, "bf16"), ["bwd"])])
    rows = [r for r in rows if "token_rows" in r["name"] or "small_dvdk" in r["name"]]
    assert any("small_dvdk_kernel" in r["name"] for r in rows) == own, rows
    assert not own or rows[-1]["grid"][0] == T, rows


# The one-launch dispatch does one workgroup's work step after step where blocks are few and tokens many: 82.6 us for a forward
# that took 71.0 with two launches (16384 tokens x 4 of 4 blocks), 69.6 / 60.2 (x 1 of 1); 58.7 / 55.3 with popular blocks
# where a block's workgroup placed all of its tokens (8192 x 8 of 24).
@pytest.mark.parametrize("T, top_e, n_blocks, form", [
    (16384, 1, 1, "place"), (16384, 4, 4, "place"), (8192, 8, 16, "place"), (8192, 2, 2, "place"), (4096, 1, 1, "one"),
    (4096, 16, 16, "one"), (4097, 1, 1, "place"), (4097, 1, 2, "few"), (8192, 8, 24, "few"), (8192, 2, 32, "few"), (8192, 2, 33, "one"),
    (16384, 4, 64, "few"), (16384, 4, 65, "one"), (16384, 1, 4, "place"), (16384, 1, 5, "few")])
def test_dispatch_of_few_blocks(T, top_e, n_blocks, form):
    for call in ("fwd", "bwd"):
        rows, = record([(shape(T, 64, n_blocks, 16, top_e, top_e, "bf16"), [call])])
        got = {"place": "dispatch_place", "few": "dispatch_one_kernelILb%dELb1E" % (call == "fwd"),
               "one": "dispatch_one_kernelILb%dELb0E" % (call == "fwd")}
        assert [f for f, name in got.items() if any(name in r["name"] for r in rows)] == [form], rows


# Grouped by five launches, 8192 pairs of 16 neurons out of 262144 took 37 us in all instead of 28 as one pass over the pairs did
# that read all rows per pair; by one launch, with dV and dK out of one kernel, 24.
@pytest.mark.parametrize("T, d, N, top_k, dtype, kernels", [
    (512, 256, 262144, 16, "bf16", ["pair_one", "seg_rows", "pair_rows"]),
    (8, 1024, 20480, 16, "f32", ["pair_one", "seg_rows", "pair_rows"]),
    (1, 16384, 262144, 16, "f32", ["pair_one", "seg_rows", "pair_rows"]),
    (1000, 768, 512, 16, "f32", ["pair_one", "seg_rows", "pair_rows"]),
    (20480, 256, 30000, 1, "f32", ["pair_one", "seg_rows", "pair_rows"]),
    (1000, 784, 4096, 16, "f32", ["pair_one", "seg_dv", "seg_dk", "pair_rows"]),
    (20481, 256, 8000, 1, "f32", ["fill_i32", "pair_count", "pair_scan", "pair_fill", "seg_sort", "seg_rows", "pair_rows"]),
    (20481, 256, 30000, 1, "f32", ["fill_i32", "pair_count", "pair_scan", "pair_fill", "seg_sort", "seg_dv", "seg_dk", "pair_rows"]),
    (64, 8, 1 << 29, 5, "f32", ["pair_one", "seg_rows", "pair_rows"]),
    (64, 8, (1 << 29) + 256, 5, "f32", ["fill_i32", "pair_count", "pair_sums", "pair_scan", "pair_fill", "seg_sort", "seg_rows", "pair_rows"])])
def test_backward_of_few_pairs(T, d, N, top_k, dtype, kernels):
    nb = 256 if N > 1 << 22 else 1
    rows, = record([(shape(T, d, nb, N // nb, 1, top_k, dtype), ["bwd"])])
    names = [r["name"] for r in rows]
    assert len(names) == len(kernels) and all(k in n for k, n in zip(kernels, names)), names


# Rows are asked for in batches of eight, whatever a token's pairs: with one pair the same row eight times (10000 tokens, d 4096,
# fp32: backward 254 us where one pass over the pairs had taken 242, 216 so).
@pytest.mark.parametrize("top_k, rows", [(1, 1), (2, 2), (3, 4), (4, 4), (5, 8), (64, 8)])
def test_rows_of_tokens_with_few_pairs(top_k, rows):
    got, = record([(shape(3000, 4096, 1, 8192, 1, top_k, "f32"), ["fwd", "bwd"])])
    names = [r["name"] for r in got if "pair_rows" in r["name"]]
    assert ["kernelIfLi%dELi%dEE" % (acc, rows) in n for acc, n in zip((1, 4), names)] == [True, True], names
