"""Components that fit in LDS: steps with at least 16 rows, 4 summed and 8 new entries multiply on the
matrix cores (few of them share their sums between waves), the others with a group of lanes per output,
and the tables of the next step are fetched during the current one, 32 step headers at a time.  Fused
programs reach the widest operators (64 x 16, 16 x 64), one step per tensor the narrow ones and more
than 32 steps.  Against the emulated program; tolerance 1e-12: the components compute in FP64."""
import numpy as np
import pytest

from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

PLAIN = jf.JF_FLAG_NO_FUSE | jf.JF_FLAG_NO_CANCEL
# qubits, gates, noise places, seed, planner flags
KEEP = jf.JF_FLAG_NO_CANCEL
CASES = [(3, 20, 2, 1, 0), (6, 80, 4, 4, 0), (4, 80, 3, 2, KEEP), (5, 80, 2, 2, KEEP), (5, 80, 3, 1, KEEP),
         (5, 120, 2, 2, KEEP), (6, 40, 3, 1, KEEP), (6, 40, 3, 2, KEEP), (6, 80, 2, 2, KEEP), (3, 12, 1, 6, PLAIN),
         (4, 60, 2, 7, PLAIN), (5, 70, 1, 8, PLAIN), (4, 90, 3, 9, PLAIN)]


def _plan(case, alg, dtype="c128"):
    n, gates, sites, seed, flags = case
    return jf.plan(gen.random_circuit(n, gates, sites, 0.01, 0.3, seed), alg, dtype, flags=flags)


def test_cases_fit_in_lds_and_reach_more_than_one_chunk_of_headers():
    plans = [_plan(c, 1) for c in CASES]
    assert all(p.info()["max_log2_intermediate"] <= 11 for p in plans)
    steps = [s for p in plans for s in p.describe()]
    wide = {(s["kS"], s["kN"], s["rC"] - s["kN"]) for s in steps if s["kS"] >= 2 and s["kN"] >= 3}
    assert {(2, 4, 4), (2, 6, 4), (4, 6, 4), (5, 5, 5), (6, 4, 4)} <= wide
    assert max(p.stats()["n_steps"] for p in plans) > 64


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_lds_components_against_emulation(case):
    p = _plan(case, 1)
    want = p.emulate()
    ws = jf.workspace(p.info()["workspace_bytes"])
    ws.fill_(255)  # NaN wherever a launch leaves something unwritten
    jf.jf_workspace_release(ws)
    for rep in range(2):
        print("[gpu-test] lds products", case, rep, flush=True)
        got = jf.jf_fidelity_alg1(p, ws, want_terms=True)
        assert np.max(np.abs(got["terms"] - want)) <= 1e-12
        assert abs(got["fj"] - np.sum(np.abs(want) ** 2)) <= 1e-11
    two = _plan(case, 2)
    if two.info()["max_log2_intermediate"] <= 11:
        assert abs(jf.jf_fidelity_alg2(two)["fj"] - got["fj"]) <= 1e-11
