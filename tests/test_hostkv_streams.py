"""Which stream the work of host-resident keys and values goes to, from the calls that the library makes of the HIP runtime
(tests/hostcalls.py): while a later layer's blocks are on their way in, the gradient rows that leave early go on another stream,
so that both use the link's two directions at once."""
import pytest

from tests.hostcalls import STREAM, record, shape

HOST_KV, KEEP_STAGED = 1, 2
DENSE = dict(T=2048, d=512, n_blocks=8, block_size=64, top_e=2, top_k=16, dtype="bf16")
PER_PAIR = dict(DENSE, dtype="f32")


def _calls(kw, flags, calls):
    return record([(shape(flags=flags, **kw), calls)])[0]


@pytest.mark.parametrize("kw", [DENSE, PER_PAIR], ids=["dense", "per_pair"])
@pytest.mark.parametrize("keep", [0, KEEP_STAGED], ids=["fetch", "kept"])
def test_gradients_do_not_queue_behind_blocks_on_their_way_in(kw, keep):
    # another layer's blocks (workspace 2) are requested, then this layer's backward runs
    rows = _calls(kw, HOST_KV | keep, ["stage2", "bwd"])
    copies = {r["stream"] for r in rows if r["what"] == "copy" and r["src"] >= 1 << 44 and r["stream"] != STREAM}
    out = [r for r in rows if r["what"] == "launch" and "rows_to_host" in r["name"]]
    assert len(copies) == 1 and len(out) == 2
    for r in out:
        assert r["stream"] not in copies
    # the caller's stream waits for whatever left on another one, after its last kernel
    side = [r["stream"] for r in out if r["stream"] != STREAM]
    if side:
        last = max(i for i, r in enumerate(rows) if r["what"] == "record" and r["stream"] == side[0])
        assert any(r["what"] == "wait" and r["stream"] == STREAM and r["event"] == rows[last]["event"] for r in rows[last:])


@pytest.mark.parametrize("kw", [DENSE, PER_PAIR], ids=["dense", "per_pair"])
def test_a_captured_backward_keeps_to_its_stream(kw):
    # the forward of the step ran eagerly; its kept copies make the backward capturable
    before = len(_calls(kw, HOST_KV | KEEP_STAGED, ["fwd"]))
    rows = _calls(kw, HOST_KV | KEEP_STAGED, ["fwd", "capture", "bwd", "no_capture"])[before:]
    assert sum("rows_to_host" in r["name"] for r in rows) == 2
    assert {r["stream"] for r in rows} == {STREAM}, rows
    assert not [r for r in rows if r["what"] == "copy"]
