"""The 64 x 128 tiles of the token-major contractions at their edges, bit for bit against the 128 x 256 tiles (which
meft_debug_global_loads forces): groups around multiples of 64 rows, blocks and hidden sizes around multiples of 64 and
128, contractions of one to a few k tiles (fewer than the ring has slots), one group for all the XCDs and more groups per
XCD than a tile search holds in registers, and blocks that leave columns of padding."""
import numpy as np
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=63, d=64, n_blocks=1, block_size=16, top_e=1, top_k=16),
    dict(T=640, d=64, n_blocks=10, block_size=130, top_e=1, top_k=9),
    dict(T=1290, d=192, n_blocks=10, block_size=126, top_e=2, top_k=30),
    dict(T=700, d=320, n_blocks=3, block_size=128, top_e=2, top_k=64),
    dict(T=1000, d=128, n_blocks=9, block_size=258, top_e=4, top_k=100, zipf_s=1.5),
    dict(T=900, d=576, n_blocks=620, block_size=48, top_e=4, top_k=20),
    dict(T=2000, d=704, n_blocks=20, block_size=72, top_e=5, top_k=60, zipf_s=0.8),
]
NAMES = ("idx", "act", "out", "dh", "dK_bits", "dV_bits", "touched")


@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_d{k['d']}_{k['n_blocks']}x{k['block_size']}_e{k['top_e']}")
def test_same_bits_as_large_tiles(kw):
    from tests import parity as P
    t = synth.make_inputs(synth.small_case(seed=6100 + kw["T"], dtype="bf16", **kw))
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


def test_a_group_of_more_than_65536_tiles():
    """One group of 65537 tiles of 64 rows: the number of a tile times the group's tiles passes 2^32."""
    import torch
    from paper_2406_04984_amd import binding as B
    T, d, bs = 65536 * 64 + 1, 64, 64
    s = B.make_shape(T, d, 1, bs, 1, 1, "bf16")
    gen = torch.Generator(device="cuda").manual_seed(6200)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    h, dOut = (torch.randn((T, d), generator=gen, **bf) for _ in range(2))
    K, V = (torch.randn((bs, d), generator=gen, **bf) for _ in range(2))
    block_idx = torch.zeros((T, 1), dtype=torch.int32, device="cuda")
    ws = torch.empty((B.meft_workspace_bytes(s),), dtype=torch.uint8, device="cuda")
    got = []
    for forced in (False, True):
        out, dh = torch.zeros((T, d), **bf), torch.zeros((T, d), **bf)
        idx, act = torch.zeros((T, 1), dtype=torch.int32, device="cuda"), torch.zeros((T, 1), device="cuda")
        dK, dV = torch.zeros((bs, d), **bf), torch.zeros((bs, d), **bf)
        touched, n = torch.zeros((bs,), dtype=torch.int32, device="cuda"), torch.zeros((1,), dtype=torch.int32, device="cuda")
        ws.fill_(0xFF)
        B.meft_debug_global_loads(forced)
        try:
            B.meft_sparse_fwd(s, h, K, V, block_idx, out, idx, act, ws)
            B.meft_sparse_bwd(s, h, K, V, idx, act, dOut, dh, dK, dV, touched, n, ws)
            torch.cuda.synchronize()
        finally:
            B.meft_debug_global_loads(False)
        got.append((idx, act, out, dh, dK, dV, touched, n))
    for x, y in zip(*got):
        assert torch.equal(x, y)
    score = h[-64:].float() @ K.float().T
    assert torch.equal(got[0][0][-64:, 0].long(), score.argmax(1))
