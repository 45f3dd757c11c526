"""The per-pair backward at its edges: hidden sizes on both sides of what a wave-per-pair kernel holds (512, 1024, 2048,
4096 columns), row ends inside a wave's columns, neurons of exactly one chunk of pairs, one more, and of several, more
neurons than a scanning workgroup counts itself, no dh."""
import pytest

from paper_2406_04984_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    dict(T=50, d=8, n_blocks=2, block_size=40, top_e=1, top_k=5, dtype="f32"),
    dict(T=260, d=520, n_blocks=3, block_size=33, top_e=2, top_k=3, dtype="f32"),
    dict(T=40, d=2048, n_blocks=2, block_size=50, top_e=2, top_k=30, dtype="f32"),
    dict(T=40, d=2056, n_blocks=2, block_size=50, top_e=2, top_k=30, dtype="f32"),
    dict(T=40, d=4096, n_blocks=2, block_size=50, top_e=2, top_k=30, dtype="f32"),
    dict(T=200, d=4096, n_blocks=1, block_size=2000, top_e=1, top_k=20, dtype="bf16"),
    dict(T=200, d=4104, n_blocks=1, block_size=2000, top_e=1, top_k=20, dtype="bf16"),
    dict(T=256, d=72, n_blocks=1, block_size=64, top_e=1, top_k=64, dtype="f32"),      # every neuron: one full chunk
    dict(T=257, d=72, n_blocks=1, block_size=64, top_e=1, top_k=64, dtype="f32"),      # every neuron: a chunk and one pair
    dict(T=700, d=136, n_blocks=1, block_size=30, top_e=1, top_k=29, dtype="f32"),
    dict(T=600, d=64, n_blocks=20, block_size=7000, top_e=2, top_k=40, dtype="f32"),   # 140000 neurons
]


@pytest.mark.parametrize("kw", CASES, ids=lambda k: f"T{k['T']}_d{k['d']}_{k['n_blocks']}x{k['block_size']}_{k['dtype']}")
def test_parity(kw):
    from tests import parity as P
    P.run_and_compare(synth.small_case(seed=7100 + kw["T"], **kw)).assert_ok()


def test_without_dh():
    import torch
    from tests import parity as P
    t = synth.make_inputs(synth.small_case(T=300, d=200, n_blocks=4, block_size=60, top_e=2, top_k=20, dtype="f32", seed=7200))
    layer = P.DeviceLayer(t)
    layer.step()
    dK, dV, touched = layer.dK.clone(), layer.dV.clone(), layer.touched.clone()
    layer.dK.zero_(); layer.dV.zero_(); layer.dh.fill_(7.0)
    layer.bwd(want_dh=False)
    torch.cuda.synchronize()
    n = int(layer.n_touched.item())
    assert torch.equal(touched[:n], layer.touched[:n])
    assert torch.equal(dK, layer.dK) and torch.equal(dV, layer.dV) and bool((layer.dh == 7.0).all())


def test_an_id_repeated_within_its_tokens():
    """Ids beyond the last neuron are clamped to it, so that a neuron may get more pairs than there are tokens."""
    import torch
    from tests import parity as P
    t = synth.make_inputs(synth.small_case(T=100, d=64, n_blocks=2, block_size=40, top_e=2, top_k=20, dtype="f32", seed=7300))
    layer = P.DeviceLayer(t)
    layer.step()
    layer.idx[:, 10:] = 80 + 5
    layer.bwd()
    torch.cuda.synchronize()
    act, dOut = layer.act.double(), layer.dOut.double()
    want = act[:, 10:].sum(1) @ dOut + ((layer.idx[:, :10] == 79) * act[:, :10]).sum(1) @ dOut
    assert torch.allclose(layer.dV[79].double(), want, rtol=1e-4, atol=1e-4 * float(want.abs().max()))
