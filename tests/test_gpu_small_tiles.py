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
