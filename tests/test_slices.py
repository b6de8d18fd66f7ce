"""Kraus-sliced plans run the variants of their first sliced level in lanes beside each other, each with
level buffers and barrier flags of its own; a workspace without room for the lanes, captured plans and
wire-sliced ones keep one lane.  Against the emulated program.  Tolerances: complex128 1e-12, complex64
1e-6 (the bars of their forms)."""
import numpy as np
import pytest

from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

TOL = {"c128": 1e-12, "c64": 1e-6}
# qubits, gates, Kraus operators per noise place, seed, bits cut from the planner's own width
CASES = [(8, 220, [4] * 6, 21, 2), (8, 220, [2] * 7, 20, 2), (8, 220, [2] * 7, 22, 2),
         (8, 220, [3] * 5, 20, 2), (9, 240, [4] * 5, 7, 3)]


def _inst(n, gates, counts, seed):
    inst = gen.random_circuit(n, gates, len(counts), 0.01, 0.3, seed)
    rng = np.random.default_rng(seed)
    for s, nk in zip(inst["noise"], counts):
        p = rng.dirichlet(np.ones(nk))
        ops = [np.sqrt(p[k]) * np.linalg.qr(rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)))[0] for k in range(nk)]
        s.pop("channel"), s.pop("p")
        s["kraus"] = [K.tolist() for K in ops]
    return inst


def _plan(case, dtype, flags=0):
    n, gates, counts, seed, cut = case
    inst = _inst(n, gates, counts, seed)
    cap = int(jf.plan(inst, 1, dtype).info()["max_log2_intermediate"]) - cut
    return jf.plan(inst, 1, dtype, max_log2=cap, flags=flags)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, [c[0], c[1], c[3], c[4], *c[2]])))
def test_sliced_plans_against_emulation(case, dtype):
    import torch
    p = _plan(case, dtype)
    assert p.stats()["n_sliced_sites"] + p.stats()["n_sliced_wires"] > 0
    want = p.emulate()
    size = p.info()["workspace_bytes"]
    lanes = p.stats()["n_sliced_wires"] == 0  # a workspace for fewer is taken
    ws = jf.workspace(size)
    ws.fill_(255)  # NaN wherever a launch leaves something unwritten
    jf.jf_workspace_release(ws)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()

    def check(what, plan, w, s):
        print("[gpu-test] slices", case, dtype, what, flush=True)
        got = jf.jf_fidelity_alg1(plan, w, s, want_terms=True)
        assert np.max(np.abs(got["terms"] - want)) <= TOL[dtype]
        assert abs(got["fj"] - np.sum(np.abs(want) ** 2)) <= 10 * TOL[dtype]

    for rep in range(2):
        check("lanes", p, ws, stream)
        check("lanes, null stream", p, ws, None)
        if lanes:
            check("one lane", p, ws[:size - 256], stream)
    g = _plan(case, dtype, jf.JF_FLAG_GRAPH)
    gws = jf.workspace(g.info()["workspace_bytes"])
    for rep in range(2):
        check("captured", g, gws, stream)
    assert jf.lib().jf_set_grid_wait(p.ptr, 0) == 0  # the barriers of every lane give up at once: run again launch by launch
    check("gave up", p, ws, stream)
    assert jf.lib().jf_set_grid_wait(p.ptr, 200000000) == 0
    check("and after", p, ws, stream)
