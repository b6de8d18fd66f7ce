"""GPU tests of grid runs: consecutive small steps executed by one launch, against the dense oracle and
against the same plan run with a launch per step (JF_FLAG_NO_CHAIN).  Tolerances: complex128 |dt| and
|dF_J| <= 1e-12, complex64 and the split form 1e-6 (the bars of their forms)."""
import sys

import numpy as np
import pytest

from oracle import dense
from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 1e-6, "bf16x6": 1e-6}
PLAIN = jf.JF_FLAG_NO_FUSE | jf.JF_FLAG_NO_CANCEL  # one step per tensor: operators from 1 x 2 to 16 x 16

# (n, gates, sites, circuit seed, flags, cap cut): LDS-only programs, tensors up to 2^12 and 2^16
# (one and several tiles a workgroup), 2^20 (runs beside larger steps), single gates (few rows,
# small operators), sliced Kraus sites, sliced wires
CASES = [(3, 40, 2, 11, 0, 0), (5, 80, 3, 12, 0, 0), (6, 90, 3, 13, 0, 0), (7, 120, 3, 14, 0, 0), (8, 160, 3, 15, 0, 0),
         (9, 250, 3, 505, 0, 0), (4, 30, 2, 16, PLAIN, 0), (6, 50, 3, 17, PLAIN, 0), (7, 60, 2, 18, PLAIN, 0),
         (6, 90, 4, 4242, 0, 3), (6, 80, 2, 700, 0, 3)]


def say(*a):
    print("[gpu-test]", *a, flush=True)
    sys.stdout.flush()


def _terms(ref):
    return np.array([ref["terms"][k] for k in sorted(ref["terms"])])


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("dtype", ["c128", "c64", "bf16x6"])
def test_grid_runs_against_oracle_and_a_launch_per_step(case, dtype):
    import torch
    n, gates, sites, seed, flags, cut = case
    inst = gen.random_circuit(n, gates, sites, 1e-3, 0.2, seed)
    ref = dense.fidelity_alg1(inst, want_terms=True)
    cap = int(jf.plan(inst, 1, dtype, flags=flags).info()["max_log2_intermediate"]) - cut if cut else 0
    side = torch.cuda.Stream()
    for alg in (1, 2) if not cut else (1,):
        p = jf.plan(inst, alg, dtype, max_log2=cap, flags=flags)
        q = jf.plan(inst, alg, dtype, max_log2=cap, flags=flags | jf.JF_FLAG_NO_CHAIN)
        g = jf.plan(inst, alg, dtype, max_log2=cap, flags=flags | jf.JF_FLAG_GRAPH)
        say("grid runs", case, "alg", alg, dtype, "steps", p.stats()["n_steps"])
        run = jf.jf_fidelity_alg1 if alg == 1 else jf.jf_fidelity_alg2
        kw = {"want_terms": True} if alg == 1 else {}
        a, b = run(p, **kw), run(q, **kw)
        assert abs(a["fj"] - ref["fj"]) <= TOL[dtype] and abs(a["fj"] - b["fj"]) <= TOL[dtype]
        if alg == 1:
            assert np.max(np.abs(a["terms"] - _terms(ref))) <= TOL[dtype]
        ws = jf.workspace(g.info()["workspace_bytes"])
        for k in range(3):  # replays, eager work between them
            assert run(g, ws, side)["fj"] == a["fj"], k
            assert run(p)["fj"] == a["fj"], k
        if p.info()["workspace_bytes"] <= jf.JF_NOALLOC_BYTES:
            assert jf.jf_fidelity_noalloc(p)["fj"] == a["fj"]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_a_grid_barrier_that_gives_up_is_run_again(dtype):
    import torch
    inst = gen.random_circuit(7, 120, 3, 1e-3, 0.2, 14)
    ref = dense.fidelity_alg1(inst, want_terms=True)
    p = jf.plan(inst, 1, dtype)
    g = jf.plan(inst, 1, dtype, flags=jf.JF_FLAG_GRAPH)
    side = torch.cuda.Stream()
    ws = jf.workspace(max(p.info()["workspace_bytes"], g.info()["workspace_bytes"], jf.jf_batch_workspace([p, g])))
    want = jf.jf_fidelity_alg1(p, ws)["fj"]
    for ticks in (0, 200000000):
        for x in (p, g):
            assert jf.lib().jf_set_grid_wait(x.ptr, ticks) == 0
        say("grid barrier wait of", ticks, "ticks", dtype)
        for _ in range(2):
            got = jf.jf_fidelity_alg1(p, ws, want_terms=True)
            assert np.max(np.abs(got["terms"] - _terms(ref))) <= TOL[dtype]
            got = jf.jf_fidelity_alg1(g, ws, side)
            assert abs(got["fj"] - ref["fj"]) <= TOL[dtype]
            assert abs(jf.jf_fidelity_noalloc(p)["fj"] - ref["fj"]) <= TOL[dtype]
            for r in jf.jf_fidelity_batch([p, g], ws, side):
                assert abs(r["fj"] - ref["fj"]) <= TOL[dtype]
            assert jf.jf_decide_equivalence(p, 1 - ref["fj"] + 0.01, ws)["decision"] == 1
    assert jf.jf_fidelity_alg1(p, ws)["fj"] == want
