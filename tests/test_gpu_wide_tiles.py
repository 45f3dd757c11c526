"""The 256 x 256 tiles of the contractions at their edges, bit for bit against the 128 x 256 tiles (which
meft_debug_global_loads forces: the same products in the same order): groups that end in a short tile of one row, of 128 rows,
one row before and after it becomes a whole one, a few rows more than a whole one; blocks and hidden sizes that leave columns of a
tile empty; one to a few k tiles (fewer than are requested ahead) in the weight gradients; fewer groups than XCDs, more than
a tile search holds in registers.  SPLIT: fewer columns of tiles than XCDs, whose tiles all XCDs have to share."""
import numpy as np
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

SPLIT = [   # every XCD's list holds every group
    dict(T=4096, d=1024, n_blocks=6, block_size=1024, top_e=3, top_k=256),    # four columns of tiles both ways
    dict(T=4100, d=1792, n_blocks=5, block_size=1792, top_e=2, top_k=100),    # seven
    dict(T=8100, d=512, n_blocks=4, block_size=512, top_e=2, top_k=128),      # two
]
CASES = [
    dict(T=97, d=512, n_blocks=16, block_size=1000, top_e=16, top_k=260),     # short tiles only, columns beyond the block
    dict(T=128, d=576, n_blocks=16, block_size=1024, top_e=16, top_k=260),    # short tiles full to the last row
    dict(T=129, d=512, n_blocks=16, block_size=1022, top_e=16, top_k=260),    # whole tiles with one row in their second half
    dict(T=223, d=704, n_blocks=18, block_size=777, top_e=18, top_k=300),     # odd rows of scores
    dict(T=257, d=2048, n_blocks=5, block_size=2560, top_e=5, top_k=250),     # split lists; a short tile of one row
    dict(T=1100, d=512, n_blocks=4, block_size=2048, top_e=4, top_k=200),     # whole tiles, then a short one, per group
    dict(T=2600, d=512, n_blocks=64, block_size=512, top_e=3, top_k=60, zipf_s=0.4),   # groups of every size
    dict(T=30000, d=512, n_blocks=600, block_size=64, top_e=3, top_k=12),     # 75 groups per XCD
    dict(T=70, d=320, n_blocks=9, block_size=200, top_e=2, top_k=24),         # weight gradients of one k tile
] + SPLIT
NAMES = ("idx", "act", "out", "dh", "dK_bits", "dV_bits", "touched")


@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_d{k['d']}_{k['n_blocks']}x{k['block_size']}_e{k['top_e']}")
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
