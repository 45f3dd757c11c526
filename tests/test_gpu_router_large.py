"""The router on either side of the lines from which its contraction runs on LDS tiles, and on more tokens than one launch
dimension can count tiles of: every token's choice against torch."""
import pytest

pytestmark = pytest.mark.gpu


SIZES = [
    (2_100_003, 8, 5, "f32"), (2_100_003, 24, 2, "bf16"),
    (3072, 512, 1024, "f32"), (3073, 512, 1024, "f32"),
    (1792, 1000, 1023, "bf16"), (1793, 1000, 1023, "bf16"),
    (910, 2056, 1024, "bf16"), (911, 2056, 1024, "bf16"),
    (10240, 2048, 5, "bf16"), (10241, 2048, 5, "bf16"),
    (12000, 2112, 3, "bf16"), (16000, 2112, 3, "bf16"),
]


@pytest.mark.parametrize("T, d, n_blocks, dtype", SIZES)
def test_choices_of_all_tokens(T, d, n_blocks, dtype):
    import torch
    from paper_2406_04984_amd import binding as B
    s = B.make_shape(T, d, n_blocks, 16, 1, 4, dtype)
    gen = torch.Generator(device="cuda").manual_seed(9100)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    # small whole numbers: scores are exact, ties go to the lower block
    h = torch.randint(-8, 9, (T, d), generator=gen, device="cuda").to(tdt)
    Wg = torch.randint(-8, 9, (n_blocks, d), generator=gen, device="cuda").to(tdt)
    idx = torch.full((T, 1), -1, dtype=torch.int32, device="cuda")
    score = torch.zeros((T, 1), device="cuda")
    ws = torch.empty((B.meft_workspace_bytes(s),), dtype=torch.uint8, device="cuda")
    B.meft_route(s, h, Wg, None, idx, score, ws)
    torch.cuda.synchronize()
    want = h.float() @ Wg.float().T
    top = want.max(1).values
    assert torch.equal(score[:, 0], top)
    first = (want == top[:, None]).int().argmax(1)
    assert torch.equal(idx[:, 0].long(), first)
