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


def test_more_tokens_than_a_launch_has_along_x():
    """2^23 + 1 tokens of whole numbers (every sum is exact): the tokens go on along y."""
    import torch
    from paper_2406_04984_amd import binding as B
    T, d, nb, bs = (1 << 23) + 1, 8, 128, 255
    N = nb * bs
    s = B.make_shape(T, d, nb, bs, 1, 1, "f32")
    gen = torch.Generator(device="cuda").manual_seed(7300)
    h, dOut, K, V = (torch.randint(-3, 4, (n, d), generator=gen, device="cuda").float() for n in (T, T, N, N))
    idx = torch.randint(0, N, (T, 1), generator=gen, device="cuda", dtype=torch.int32)
    act = torch.randint(0, 3, (T, 1), generator=gen, device="cuda").float()
    dh, dK, dV = torch.full((T, d), 7.0, device="cuda"), torch.zeros((N, d), device="cuda"), torch.zeros((N, d), device="cuda")
    touched, n = torch.zeros((N,), dtype=torch.int32, device="cuda"), torch.zeros((1,), dtype=torch.int32, device="cuda")
    ws = torch.empty((B.meft_workspace_bytes(s),), dtype=torch.uint8, device="cuda")
    B.meft_sparse_bwd(s, h, K, V, idx, act, dOut, dh, dK, dV, touched, n, ws)
    torch.cuda.synchronize()
    j = idx[:, 0].long()
    ds = (dOut * V[j]).sum(1, keepdim=True) * (act > 0)
    assert torch.equal(dh, ds * K[j])
    assert torch.equal(dV, torch.zeros_like(dV).index_add_(0, j, act * dOut))
    assert torch.equal(dK, torch.zeros_like(dK).index_add_(0, j, ds * h))
    ids = torch.unique(j)
    assert int(n) == len(ids) and torch.equal(touched[:len(ids)].long(), ids)
