"""The 256 x 256 tiles of the contractions at their edges, bit for bit against the 128 x 256 tiles (which
meft_debug_global_loads forces: the same products in the same order).  EDGES: groups of given sizes, one block per token; `wide` says
which contractions of a step run on such tiles (test_kernels_chosen.py holds them to it).  SPLIT: routed, fewer groups than XCDs and
fewer columns of tiles, which all XCDs have to share."""
import numpy as np
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

SCORES, MASKED, VALUES, GRADIENTS, ALONE = "ProbTokKCILi3E", "ProbTokKCILi1E", "ProbTokNC", "ProbNeuTN", "ProbTokKCILi0E"
EDGES = [   # (sizes, taken in turn by the blocks; the shape; wide)
    # whole tiles only, one row into a short tile, one row into and out of a tile's second half; one k tile more than are requested ahead
    ([257, 512, 513, 256, 768, 640, 641, 511], dict(d=512, n_blocks=32, block_size=1024, top_k=64), (VALUES, GRADIENTS)),
    # columns of tiles left empty by the hidden size and by the block, rows of scores of an odd length
    ([300, 129, 257, 640], dict(d=704, n_blocks=32, block_size=777, top_k=64), (SCORES, MASKED, VALUES)),
    # short tiles alone, of one row and full to the last one
    ([1, 128, 127, 110, 120, 128, 90, 128], dict(d=2048, n_blocks=128, block_size=520, top_k=64), (SCORES, MASKED, VALUES)),
    # 75 groups per XCD, more than a tile search holds in registers: two loads of the list, and back for the cursor behind
    ([96, 128, 129, 65, 200, 256, 17, 140], dict(d=512, n_blocks=600, block_size=450, top_k=32), (SCORES, MASKED, VALUES, GRADIENTS)),
    # lists that every XCD holds: a short tile of one row per group, and none
    ([2049, 1921, 1920, 2305], dict(d=1088, n_blocks=5, block_size=1000, top_k=64), (SCORES, MASKED, VALUES)),
    # weight gradients of one to four k tiles, behind groups that are summed pair by pair
    ([1, 17, 64, 65, 63, 130, 192, 40], dict(d=512, n_blocks=96, block_size=1024, top_k=32), (GRADIENTS,)),
    # scores alone, the rest pair by pair
    ([129, 257, 300, 385], dict(d=704, n_blocks=9, block_size=4096, top_k=32), (ALONE,)),
]
SPLIT = [   # every XCD's list holds every group
    dict(T=4096, d=1024, n_blocks=6, block_size=1024, top_e=3, top_k=256),    # four columns of tiles both ways
    dict(T=4100, d=1792, n_blocks=5, block_size=1792, top_e=2, top_k=100),    # seven
    dict(T=8100, d=512, n_blocks=4, block_size=512, top_e=2, top_k=128),      # two
]
ROUTED = SPLIT + [dict(T=2600, d=512, n_blocks=64, block_size=512, top_e=3, top_k=60, zipf_s=0.4)]   # groups of every size
NAMES = ("idx", "act", "out", "dh", "dK_bits", "dV_bits", "touched")


def group_sizes(sizes, n_blocks):
    return [sizes[i % len(sizes)] for i in range(n_blocks)]


@pytest.mark.parametrize("kw", ROUTED, ids=lambda k: f"T{k['T']}_d{k['d']}_{k['n_blocks']}x{k['block_size']}_e{k['top_e']}")
def test_same_bits_as_tiles_of_128_rows(kw):
    from tests import parity as P
    t = synth.make_inputs(synth.small_case(seed=6300 + kw["T"], dtype="bf16", **kw))
    layer = P.DeviceLayer(t)
    got = []
    for forced in (False, True):
        layer.fill_grad_sentinel()
        layer.ws.fill_(0xFF)
        layer.B.meft_debug_global_loads(forced)
        try:
            layer.step()
            got.append(layer.results())
        finally:
            layer.B.meft_debug_global_loads(False)
    for n in NAMES:
        assert np.array_equal(got[0][n], got[1][n]), n


@pytest.mark.parametrize("sizes, kw, wide", EDGES, ids=lambda v: f"d{v['d']}_{v['n_blocks']}x{v['block_size']}" if isinstance(v, dict) else "")
def test_same_bits_with_groups_of_given_sizes(sizes, kw, wide):
    import torch
    from paper_2406_04984_amd import binding as B
    rows = group_sizes(sizes, kw["n_blocks"])
    T, d, N, k = sum(rows), kw["d"], kw["n_blocks"] * kw["block_size"], kw["top_k"]
    s = B.make_shape(T, d, kw["n_blocks"], kw["block_size"], 1, k, "bf16")
    gen = torch.Generator(device="cuda").manual_seed(6500 + T)
    bf, i32 = dict(dtype=torch.bfloat16, device="cuda"), dict(dtype=torch.int32, device="cuda")
    h, dOut = (torch.randn((T, d), generator=gen, **bf) for _ in range(2))
    K, V = (torch.randn((N, d), generator=gen, **bf) / d ** 0.5 for _ in range(2))
    blocks = torch.arange(kw["n_blocks"], **i32).repeat_interleave(torch.tensor(rows, device="cuda"))
    blocks = blocks[torch.randperm(T, generator=gen, device="cuda")].reshape(T, 1).contiguous()
    ws = torch.empty((B.meft_workspace_bytes(s),), dtype=torch.uint8, device="cuda")
    got = []
    for forced in (False, True):
        out, dh = torch.zeros((T, d), **bf), torch.zeros((T, d), **bf)
        dK, dV = torch.zeros((N, d), **bf), torch.zeros((N, d), **bf)
        idx, act = torch.full((T, k), -1, **i32), torch.zeros((T, k), dtype=torch.float32, device="cuda")
        touched, n_touched = torch.full((min(N, T * k),), -1, **i32), torch.zeros((1,), **i32)
        ws.fill_(0xFF)
        B.meft_debug_global_loads(forced)
        try:
            B.meft_sparse_fwd(s, h, K, V, blocks, out, idx, act, ws)
            ws.fill_(0xFF)
            B.meft_sparse_bwd(s, h, K, V, idx, act, dOut, dh, dK, dV, touched, n_touched, ws)
            torch.cuda.synchronize()
        finally:
            B.meft_debug_global_loads(False)
        assert out.abs().max() > 0 and dh.abs().max() > 0 and dK.abs().max() > 0 and dV.abs().max() > 0
        got.append((idx, act, out, dh, dK, dV, touched, n_touched))
    for x, y in zip(*got):
        assert torch.equal(x, y)
