"""Which small steps run several to a launch (host only): all that may where no chain competes, and not the
steps of long chains of FP32 or split steps, whose one launch is cheaper than their exchanges."""
import pytest

from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

QUICK = jf.JF_FLAG_EFFORT(1)


def _small(s):
    lim = {"c64": 17, "c128": 16}
    return s["rA"] <= lim[s["in_prec"]] and s["rC"] <= lim[s["out_prec"]] and s["kS"] + s["kN"] <= 10


def _circuits():
    for n, gates, sites in ((7, 300, 5), (7, 150, 3), (8, 220, 3), (9, 250, 3)):
        yield gen.random_circuit(n, gates, sites, 1e-3, 1e-2, 22)


@pytest.mark.parametrize("alg", [1, 2])
def test_complex128_steps_join_runs_wherever_they_may(alg):
    for inst in _circuits():
        steps = jf.plan(inst, alg, "c128", flags=QUICK).describe()
        for a, b in zip(steps, steps[1:]):  # neighbours that may, in runs of at most 48
            if _small(a) and _small(b):
                assert a["run"] >= 0 and b["run"] >= 0
        assert not any(s["run"] >= 0 and not _small(s) for s in steps)


@pytest.mark.parametrize("dtype", ["c64", "bf16x6"])
@pytest.mark.parametrize("alg", [1, 2])
def test_long_chains_keep_their_launch(alg, dtype):
    left = 0
    for inst in _circuits():
        p = jf.plan(inst, alg, dtype, flags=QUICK)
        steps = p.describe()
        chains = {}
        for s in steps:
            if s["chain"] >= 0:
                chains.setdefault((s["comp"], s["chain"]), []).append(s)
        for chain in chains.values():
            if len(chain) >= 3 and chain[0]["compute"] == "f32" and chain[0]["rA"] >= 12 and _small(chain[0]):
                assert all(s["run"] < 0 for s in chain) or chain[0]["rA"] < 14
                left += all(s["run"] < 0 for s in chain)
        runs = {}
        for i, s in enumerate(steps):
            if s["run"] >= 0:
                runs.setdefault((s["comp"], s["run"]), []).append(i)
        for at in runs.values():
            assert 2 <= len(at) <= 48 and at == list(range(at[0], at[0] + len(at)))
            # a run never starts inside a chain that is launched
            s = steps[at[0]]
            if s["chain"] >= 0 and at[0] and steps[at[0] - 1]["chain"] == s["chain"]:
                assert steps[at[0] - 1]["run"] >= 0
    assert dtype != "c64" or left > 0
