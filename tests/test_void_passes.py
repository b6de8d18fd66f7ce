"""GPU tests of passes whose grid barrier gives up: with a wait of 0 every workgroup leaves at its first
barrier, and the result has to come from the pass that is run again with a launch per step, also on a
plan, a workspace and a landing area that no pass has written before (a stale answer cannot pass).
Tolerances: complex128 1e-12, complex64 and the split form 1e-6 (the bars of their forms)."""
import numpy as np
import pytest

from oracle import dense
from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 1e-6, "bf16x6": 1e-6}
QUICK = jf.JF_FLAG_EFFORT(1)  # little path search
PLAIN = QUICK | jf.JF_FLAG_NO_FUSE | jf.JF_FLAG_NO_CANCEL  # one step per tensor: more than one run of small steps
CASES = {"one run": (8, 220, 3, 22, QUICK), "several runs": (7, 60, 2, 18, PLAIN)}
DEFAULT_WAIT = 200000000


def _case(name):
    n, gates, sites, seed, flags = CASES[name]
    inst = gen.random_circuit(n, gates, sites, 1e-3, 0.2, seed)
    ref = dense.fidelity_alg1(inst, want_terms=True)
    return inst, flags, ref["fj"], np.array([ref["terms"][k] for k in sorted(ref["terms"])])


def _workspace(nbytes):
    import torch
    ws = jf.workspace(nbytes)
    ws.fill_(255)  # NaN wherever a launch leaves something unwritten
    jf.jf_workspace_release(ws)
    torch.cuda.synchronize()
    return ws


def _never_waits(p):
    assert jf.lib().jf_set_grid_wait(p.ptr, 0) == 0
    return p


def _run(p, alg, ws, stream=None):
    return jf.jf_fidelity_alg1(p, ws, stream, want_terms=True) if alg == 1 else jf.jf_fidelity_alg2(p, ws, stream)


@pytest.mark.parametrize("dtype", ["c128", "c64", "bf16x6"])
@pytest.mark.parametrize("name", CASES)
def test_a_first_pass_whose_barrier_gives_up(name, dtype):
    import torch
    inst, flags, fj, terms = _case(name)
    side = torch.cuda.Stream()
    for alg in (1, 2):
        for graph in (0, jf.JF_FLAG_GRAPH):
            print("[gpu-test] void pass", name, dtype, "alg", alg, "graph", bool(graph), flush=True)
            p = _never_waits(jf.plan(inst, alg, dtype, flags=flags | graph))
            ws = _workspace(p.info()["workspace_bytes"])
            got = _run(p, alg, ws, side if graph else None)
            assert p.last_pass()["reruns"] == 1
            assert abs(got["fj"] - fj) <= TOL[dtype]
            if alg == 1:
                assert np.max(np.abs(got["terms"] - terms)) <= TOL[dtype]


@pytest.mark.parametrize("name", CASES)
def test_a_void_pass_on_the_shared_scratch(name):
    """The scratch of jf_fidelity_noalloc holds another plan's result when the barrier gives up."""
    inst, flags, fj, terms = _case(name)
    other = jf.plan(gen.random_circuit(8, 220, 3, 1e-3, 0.2, 20), 1, "c128", flags=QUICK)
    p = _never_waits(jf.plan(inst, 1, "c128", flags=flags))
    print("[gpu-test] void pass without allocations", name, flush=True)
    jf.jf_fidelity_noalloc(other)
    got = jf.jf_fidelity_noalloc(p, want_terms=True)
    assert p.last_pass()["reruns"] == 1
    assert abs(got["fj"] - fj) <= 1e-12 and np.max(np.abs(got["terms"] - terms)) <= 1e-12


def test_void_passes_in_a_batch_and_a_decision():
    import torch
    cases = [_case(name) for name in CASES]
    for stream in (torch.cuda.Stream(), None):
        print("[gpu-test] void passes in a batch", "stream" if stream else "null", flush=True)
        plans = [_never_waits(jf.plan(c[0], 1, "c128", flags=c[1])) for c in cases]
        ws = _workspace(jf.jf_batch_workspace(plans))
        for p, c, r in zip(plans, cases, jf.jf_fidelity_batch(plans, ws, stream)):
            assert p.last_pass()["reruns"] == 1 and abs(r["fj"] - c[2]) <= 1e-12
    inst, flags, fj, _ = cases[0]
    p = _never_waits(jf.plan(inst, 1, "c128", flags=flags))
    print("[gpu-test] void pass of a decision", flush=True)
    d = jf.jf_decide_equivalence(p, 1 - fj + 0.01, _workspace(p.info()["workspace_bytes"]))
    assert p.last_pass()["reruns"] == 1 and d["decision"] == 1 and abs(d["fj_lower"] - fj) <= 1e-12


def test_entries_of_one_plan_in_a_batch_have_a_result_each():
    """A plan that stands in a batch twice: each entry's give-up is seen and its pass run again."""
    import torch
    inst, flags, fj, _ = _case("one run")
    for graph_stream in (torch.cuda.Stream(), None):
        p = jf.plan(inst, 1, "c128", flags=flags)
        q = jf.plan(gen.random_circuit(8, 220, 3, 1e-3, 0.2, 20), 1, "c128", flags=QUICK)
        want = jf.jf_fidelity_alg1(q)["fj"]
        batch = [p, q, p, p]
        ws = _workspace(jf.jf_batch_workspace(batch))
        for wait, reruns in ((0, 3), (DEFAULT_WAIT, 0)):
            assert jf.lib().jf_set_grid_wait(p.ptr, wait) == 0
            for rep in range(2):
                print("[gpu-test] a plan three times in a batch, wait", wait, "rep", rep, flush=True)
                got = [r["fj"] for r in jf.jf_fidelity_batch(batch, ws, graph_stream)]
                assert (rep or p.last_pass()["reruns"] == reruns) and q.last_pass()["reruns"] == 0
                assert max(abs(g - w) for g, w in zip(got, (fj, want, fj, fj))) <= 1e-12


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_a_run_that_gives_up_while_it_is_timed_is_not_taken(dtype):
    """Tuning: the launches after a give-up end at once, which must not read as fast, neither for the plan
    nor for others of its shape."""
    inst, flags, fj, _ = _case("one run")
    p = _never_waits(jf.plan(inst, 1, dtype, flags=flags))
    ws = _workspace(p.info()["workspace_bytes"])
    print("[gpu-test] tuning without waits", dtype, flush=True)
    jf.jf_autotune(p, ws)
    got = jf.jf_fidelity_alg1(p, ws)
    assert p.last_pass()["reruns"] == 0 and p.last_pass()["grid_launches"] == 0 and abs(got["fj"] - fj) <= TOL[dtype]
    q = jf.plan(inst, 1, dtype, flags=flags)
    print("[gpu-test] tuning with waits", dtype, flush=True)
    jf.jf_autotune(q, ws)
    got = jf.jf_fidelity_alg1(q, ws)
    assert q.last_pass()["reruns"] == 0 and q.last_pass()["grid_launches"] > 0 and abs(got["fj"] - fj) <= TOL[dtype]


@pytest.mark.parametrize("name", CASES)
def test_a_barrier_that_gave_up_is_not_waited_for_again(name):
    """After a give-up the plan's passes go out launch by launch, until it is let try again."""
    import torch
    inst, flags, fj, _ = _case(name)
    side = torch.cuda.Stream()
    for way in ("eager", "graph", "scratch", "batch", "batch, null stream"):
        p = jf.plan(inst, 1, "c128", flags=flags | (jf.JF_FLAG_GRAPH if way == "graph" else 0))
        ws = _workspace(jf.jf_batch_workspace([p]))
        run = {"eager": lambda: jf.jf_fidelity_alg1(p, ws), "graph": lambda: jf.jf_fidelity_alg1(p, ws, side),
               "scratch": lambda: jf.jf_fidelity_noalloc(p), "batch": lambda: jf.jf_fidelity_batch([p], ws, side)[0],
               "batch, null stream": lambda: jf.jf_fidelity_batch([p], ws, None)[0]}[way]
        for again in ("wait", "kernel choice"):
            _never_waits(p)
            for reruns in (1, 0, 0):
                print("[gpu-test] launch by launch after a give-up", name, way, "reruns", reruns, flush=True)
                assert abs(run()["fj"] - fj) <= 1e-12
                assert p.last_pass()["reruns"] == reruns and p.last_pass()["grid_launches"] == 0
            if again == "kernel choice":  # tries, and gives up at the wait of 0
                jf.jf_set_kernel_variant(p, jf.KV_AUTO)
                assert abs(run()["fj"] - fj) <= 1e-12 and p.last_pass()["reruns"] == 1
            assert jf.lib().jf_set_grid_wait(p.ptr, DEFAULT_WAIT) == 0
            print("[gpu-test] and with its wait again", flush=True)
            assert abs(run()["fj"] - fj) <= 1e-12
            assert p.last_pass()["reruns"] == 0 and p.last_pass()["grid_launches"] > 0
