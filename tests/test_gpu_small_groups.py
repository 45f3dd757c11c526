"""Unbalanced routing on the block-dense path (the paper trains its router without a balancing loss, Section 3.2, so
some blocks receive a handful of tokens): groups of at most min(16, top_e * block_size / top_k) tokens are taken out
of the matrix-core contractions that follow the selection and computed pair by pair.  Group sizes on both sides of
that limit, in one batch, with the forward's tables reused by the backward and without; same parity rules as
everywhere else."""
import numpy as np
import pytest

from paper_2406_04984_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


def _assigned(cfg, loads, seed):
    """Inputs whose router sends exactly loads[b] tokens to block b first (tokens in a seeded order): the hidden
    states carry a strong component along one of n_blocks orthonormal directions, which are the router's rows."""
    assert sum(loads) == cfg.T and len(loads) == cfg.n_blocks <= cfg.d
    t = synth.make_inputs(cfg)
    rng = np.random.default_rng(seed)
    q, _ = np.linalg.qr(rng.standard_normal((cfg.d, cfg.n_blocks)))
    dirs = q.T.astype(np.float32)                                   # [n_blocks, d], orthonormal rows
    first = rng.permutation(np.repeat(np.arange(cfg.n_blocks), loads))
    t.Wg = dirs.copy()
    t.h = t.h + 12.0 * dirs[first]
    t.bias = None
    if cfg.dtype == "bf16":
        t.h = synth.bf16_to_f32(synth.bf16_round(t.h))
        t.Wg = synth.bf16_to_f32(synth.bf16_round(t.Wg))
    return t, first


def _check(t, rows=None):
    from oracle import oracle
    cfg = t.cfg
    g = P.run_gpu(t)
    r = oracle.route(t.h, t.Wg, cfg.top_e, t.bias)
    f = oracle.forward(t.h, t.K, t.V, r.block_idx, cfg.block_size, cfg.top_k, want_candidates=True)
    rep = P.compare(t, g, r, f, None)
    print(rep.summary(), flush=True)
    rep.assert_ok()
    again = P.run_gpu(t)
    for n in ("idx", "out", "dK_bits", "dV_bits", "dh", "touched"):
        assert np.array_equal(g[n], again[n]), n
    return g


LOADS = [0, 1, 2, 7, 8, 9, 15, 16, 17, 18, 33, 130, 0, 200, 16, 5]      # 16 blocks


@pytest.mark.parametrize("top_k", [9, 4], ids=["limit8", "limit16"])
@pytest.mark.parametrize("reuse", [True, False], ids=["reuse_fwd", "rebuild"])
def test_group_sizes_around_the_limit_one_block_per_token(reuse, top_k):
    cfg = synth.small_case(T=sum(LOADS), d=192, n_blocks=len(LOADS), block_size=72, top_e=1, top_k=top_k,
                           dtype="bf16", seed=1401, reuse_fwd=reuse)
    t, first = _assigned(cfg, LOADS, seed=3)
    g = _check(t)
    assert np.array_equal(np.bincount(g["block_idx"].ravel(), minlength=cfg.n_blocks), LOADS)


@pytest.mark.parametrize("reuse", [True, False], ids=["reuse_fwd", "rebuild"])
def test_group_sizes_around_the_limit_three_blocks_per_token(reuse):
    # the first block of every token is assigned, the other two follow the noise: every block also collects
    # some tokens through those, so the sizes are checked to lie on both sides of the limit rather than fixed
    cfg = synth.small_case(T=sum(LOADS), d=256, n_blocks=len(LOADS), block_size=64, top_e=3, top_k=24, dtype="bf16",
                           seed=1402, reuse_fwd=reuse)
    t, _ = _assigned(cfg, LOADS, seed=4)
    t.bias = np.where(np.arange(cfg.n_blocks) < 8, -3.0, 0.0).astype(np.float32)   # keeps blocks 0..7 nearly empty
    g = _check(t)
    sizes = np.bincount(g["block_idx"].ravel(), minlength=cfg.n_blocks)
    assert (sizes[sizes > 0] <= 8).sum() >= 3 and (sizes > 8).sum() >= 3, sizes


@pytest.mark.parametrize("T, n_blocks, reuse", [(96, 40, True), (300, 200, True), (300, 200, False)],
                         ids=["few_tokens", "reuse_fwd", "rebuild"])
def test_every_group_is_small(T, n_blocks, reuse):
    # more blocks than tokens per block: no group reaches the matrix cores after the selection
    cfg = synth.small_case(T=T, d=128, n_blocks=n_blocks, block_size=32, top_e=2, top_k=4, dtype="bf16", seed=1403,
                           reuse_fwd=reuse)
    g = _check(synth.make_inputs(cfg))
    assert np.bincount(g["block_idx"].ravel(), minlength=cfg.n_blocks).max() <= 16


def test_zipf_loads_wide_hidden_size():
    # hidden size of two 8-element vectors per thread; loads from a Zipf-like router bias
    cfg = synth.small_case(T=700, d=4096, n_blocks=48, block_size=64, top_e=2, top_k=16, dtype="bf16", seed=1404,
                           zipf_s=1.2, reuse_fwd=True)
    g = _check(synth.make_inputs(cfg))
    sizes = np.bincount(g["block_idx"].ravel(), minlength=cfg.n_blocks)
    assert (sizes[sizes > 0] <= 8).sum() >= 3 and (sizes > 8).sum() >= 3, sizes


def test_backward_without_dh_leaves_it_alone():
    cfg = synth.small_case(T=sum(LOADS), d=192, n_blocks=len(LOADS), block_size=72, top_e=1, top_k=9, dtype="bf16",
                           seed=1405, reuse_fwd=True)
    t, _ = _assigned(cfg, LOADS, seed=5)
    ref = P.run_gpu(t)
    layer = P.DeviceLayer(t)
    layer.fill_grad_sentinel()
    layer.route()
    layer.fwd()
    layer.dh.fill_(7.0)
    layer.bwd(want_dh=False)
    got = layer.results()
    for n in ("idx", "act", "out", "dK_bits", "dV_bits", "touched"):
        assert np.array_equal(ref[n], got[n]), n
    assert bool((layer.dh == 7.0).all())


@pytest.mark.parametrize("T, d", [(200, 1024), (4100, 64)], ids=["columns_shared", "token_per_workgroup"])
def test_lists_of_pairs_in_several_pieces(T, d):
    # 1500 of 3000 candidates: a token's pairs of small groups (at most two tokens) are listed 1024 positions at a time
    cfg = synth.small_case(T=T, d=d, n_blocks=60, block_size=1000, top_e=3, top_k=1500, dtype="bf16", seed=1406, zipf_s=2.5,
                           reuse_fwd=True)
    g = _check(synth.make_inputs(cfg))
    sizes = np.bincount(g["block_idx"].ravel(), minlength=cfg.n_blocks)
    assert ((sizes > 0) & (sizes <= 2)).sum() >= 2, sizes
