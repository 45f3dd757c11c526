"""meft_debug_global_loads from another host thread during a call: a batch-union call's launches depend on each other's choice of
loads (rows gathered by the contractions, or compacted first), so a call is made of the launches that one choice gives, wherever
in the call the other thread comes."""
import pytest

from tests.hostcalls import record, shape

UNION = shape(1700, 512, 1, 5000, 1, 8, "bf16")   # large tiles: the rows are gathered by the contractions


@pytest.mark.parametrize("call", ["union_fwd", "union_bwd"])
def test_one_choice_of_loads_per_call(call):
    names = lambda rows: [r["name"] for r in rows if r["what"] == "launch"]
    whole = names(record([(UNION, [call])])[0])
    assert any("ProbTokNCRows" in n for n in whole) and not any("gather_rows" in n for n in whole), whole
    flipped = record([(UNION, [f"flip {n}", call]) for n in range(1, len(whole) + 1)])
    for n, rows in enumerate(flipped, 1):
        assert names(rows) == whole, n
