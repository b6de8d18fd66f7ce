"""What a plan asks for as its workspace (host only)."""
import pytest

from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

QUICK = jf.JF_FLAG_EFFORT(1)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_captured_plans_ask_for_one_lane(dtype):
    """The slices of a captured plan run one after another, so its workspace holds one lane's buffers."""
    inst = gen.random_circuit(8, 220, 6, 0.01, 0.3, 21)
    cap = int(jf.plan(inst, 1, dtype, flags=QUICK).info()["max_log2_intermediate"]) - 2
    p = jf.plan(inst, 1, dtype, max_log2=cap, flags=QUICK)
    g = jf.plan(inst, 1, dtype, max_log2=cap, flags=QUICK | jf.JF_FLAG_GRAPH)
    assert p.stats()["n_sliced_sites"] > 0 and p.stats()["n_sliced_wires"] == 0
    steps = p.describe()
    assert [s["rC"] for s in steps] == [s["rC"] for s in g.describe()]
    # a lane's two buffers of the widest level: four lanes against one
    widest = (8 if dtype == "c64" else 16) << max(s["rC"] for s in steps)
    assert p.info()["workspace_bytes"] - g.info()["workspace_bytes"] >= 3 * 2 * widest
    # and without the slices, as much as the same plan uncaptured
    p, g = (jf.plan(inst, 1, dtype, flags=QUICK | f) for f in (0, jf.JF_FLAG_GRAPH))
    assert p.info()["workspace_bytes"] == g.info()["workspace_bytes"]
