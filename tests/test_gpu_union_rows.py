"""Batch union with K's and V's rows gathered by the contractions, bit for bit against compacted copies (which
meft_debug_global_loads forces): unions that end inside a k tile, inside a column tile, with a virtual block and one row behind it,
virtual blocks that are no multiple of a column tile, hidden sizes that are none, one and several virtual blocks, and rows outside
the union that hold no numbers, which nothing may touch.  SMALL: on small tiles, which read compacted copies either way."""
import pytest

pytestmark = pytest.mark.gpu

GATHERED = [  # T, d, N, neurons in the union, top_k
    (1700, 512, 5000, 3111, 8), (2100, 1024, 4096, 4096, 4),
    (8100, 960, 900, 801, 4), (2100, 960, 1500, 1025, 4), (8100, 448, 2000, 1999, 2), (1100, 2048, 24576, 20001, 20),
]
SMALL = [(1500, 4096, 2048, 1025, 16), (9000, 320, 1300, 1100, 3)]


@pytest.mark.parametrize("T, d, N, U, k", GATHERED + SMALL, ids=lambda v: str(v))
def test_same_bits_as_compacted_copies(T, d, N, U, k):
    import torch
    from paper_2406_04984_amd import binding as B
    s = B.make_shape(T, d, 1, N, 1, k, "bf16")
    gen = torch.Generator(device="cuda").manual_seed(8600 + T)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    h, dOut = (torch.randn((T, d), generator=gen, **bf) for _ in range(2))
    K, V = (torch.randn((N, d), generator=gen, **bf) / d ** 0.5 for _ in range(2))
    rows = torch.randperm(N, generator=gen, device="cuda")[:U].sort()[0]
    unused = torch.ones(N, dtype=torch.bool, device="cuda")
    unused[rows] = False
    K[unused], V[unused] = float("nan"), float("inf")
    # every neuron of the union is selected by some token
    pick = rows[torch.arange(T * k, device="cuda") % U].reshape(T, k).sort(1)[0].to(torch.int32)
    ws = torch.empty((B.meft_union_workspace_bytes(s),), dtype=torch.uint8, device="cuda")
    got = []
    for forced in (False, True):
        out, dh = torch.zeros((T, d), **bf), torch.zeros((T, d), **bf)
        dK, dV = torch.zeros((N, d), **bf), torch.zeros((N, d), **bf)
        S, n = torch.zeros((min(N, T * k),), dtype=torch.int32, device="cuda"), torch.zeros((1,), dtype=torch.int32, device="cuda")
        ws.fill_(0xFF)
        B.meft_debug_global_loads(forced)
        try:
            B.meft_union_fwd(s, h, K, V, pick, out, S, n, ws)
            ws.fill_(0xFF)
            B.meft_union_bwd(s, h, K, V, S, n, dOut, dh, dK, dV, ws)
            torch.cuda.synchronize()
        finally:
            B.meft_debug_global_loads(False)
        assert int(n) == U and torch.equal(S[:U].long(), rows)
        assert torch.isfinite(out.float()).all() and torch.isfinite(dh.float()).all() and out.abs().max() > 0
        got.append((out, dh, dK, dV))
    for x, y in zip(*got):
        assert torch.equal(x, y)
