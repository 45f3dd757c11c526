"""The forward of a few tokens and the untiled router scores, at the edges of their tiles: token groups around 16 and 32,
block sizes that are no multiple of 16 or 4, hidden sizes whose rows end inside a 64-byte step, fewer and more entries
than blocks, the largest batch that takes this path and the first that does not, selection only, and a backward that is
told to reuse tables this forward does not leave."""
import numpy as np
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=1, d=8, n_blocks=1, block_size=1, top_e=1, top_k=1, dtype="f32"),
    dict(T=1, d=4096, n_blocks=70, block_size=130, top_e=5, top_k=100, dtype="bf16"),
    dict(T=17, d=72, n_blocks=3, block_size=33, top_e=2, top_k=20, dtype="f32"),
    dict(T=33, d=200, n_blocks=2, block_size=50, top_e=1, top_k=50, dtype="bf16"),
    dict(T=64, d=136, n_blocks=16, block_size=47, top_e=8, top_k=300, dtype="bf16"),       # 512 entries
    dict(T=65, d=136, n_blocks=16, block_size=47, top_e=8, top_k=300, dtype="bf16"),       # one token too many
    dict(T=100, d=1032, n_blocks=300, block_size=24, top_e=3, top_k=9, dtype="f32", zipf_s=2.0),
    dict(T=128, d=64, n_blocks=1100, block_size=16, top_e=4, top_k=32, dtype="bf16"),
    dict(T=40, d=640, n_blocks=9, block_size=1024, top_e=9, top_k=1000, dtype="bf16"),
]


@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_d{k['d']}_{k['n_blocks']}x{k['block_size']}_{k['dtype']}")
def test_parity(kw):
    from tests import parity as P
    cfg = synth.small_case(seed=4100 + kw["T"], reuse_fwd=True, **kw)
    P.run_and_compare(cfg).assert_ok()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_selection_only(dtype):
    import torch
    from tests import parity as P
    t = synth.make_inputs(synth.small_case(T=20, d=256, n_blocks=12, block_size=96, top_e=3, top_k=40, dtype=dtype, seed=4200))
    layer = P.DeviceLayer(t)
    layer.route()
    layer.fwd()
    idx, act = layer.idx.clone(), layer.act.clone()
    layer.idx.fill_(-1)
    layer.B.meft_sparse_fwd(layer.shape, layer.h, layer.K, layer.V, layer.block_idx, None, layer.idx, layer.act, layer.ws)
    torch.cuda.synchronize()
    assert torch.equal(idx, layer.idx) and torch.equal(act, layer.act)


@pytest.mark.parametrize("T, n_blocks, dtype", [(15, 16, "bf16"), (1000, 63, "f32"), (4097, 64, "bf16"), (500, 257, "bf16"),
                                                (130, 1024, "f32"), (70, 1025, "bf16")])
def test_router(T, n_blocks, dtype):
    from tests import parity as P
    cfg = synth.small_case(T=T, d=320, n_blocks=n_blocks, block_size=16, top_e=min(6, n_blocks), top_k=8, dtype=dtype,
                           seed=4300 + n_blocks, zipf_s=0.7)
    P.run_and_compare(cfg).assert_ok()


@pytest.mark.parametrize("T", [2048, 2049])
def test_router_of_many_blocks_and_rounds(T):
    """Both sides of the line between keys in registers, sixteen per lane, and keys in LDS."""
    from tests import parity as P
    cfg = synth.small_case(T=T, d=64, n_blocks=1000, block_size=4, top_e=8, top_k=4, dtype="f32", seed=4400, zipf_s=0.7)
    P.run_and_compare(cfg).assert_ok()
