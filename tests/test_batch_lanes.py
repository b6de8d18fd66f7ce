"""Members of a batch run in lanes beside each other (captured graphs on a stream, launches on the null
stream), small components of all members in one launch, and one launch assembles the members that have
some.  Batches of every mix against the members' own runs, in a workspace
that holds all lanes and in one that is too small for them.  Tolerances: complex128 1e-12, complex64
1e-6 (the bars of their forms)."""
import pytest

from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

TOL = {"c128": 1e-12, "c64": 1e-6}


def _apart(a, b):
    """Two circuits on disjoint qubits."""
    inst = {"n": a["n"] + b["n"], "gates": list(a["gates"]), "noise": list(a["noise"])}
    inst["gates"] += [[g[0], [q + a["n"] for q in g[1]], g[2]] for g in b["gates"]]
    inst["noise"] += [dict(s, after=s["after"] + len(a["gates"]), qubit=s["qubit"] + a["n"]) for s in b["noise"]]
    return inst


def _rand(n, gates, sites, seed):
    return gen.random_circuit(n, gates, sites, 1e-3, 1e-2, seed)


def _members(kind):
    small = [_rand(3, 20, 2, 10 + k) for k in range(3)]
    medium = [_rand(8 + k % 2, 230, 2 + k % 3, 20 + k) for k in range(6)]
    mixed = [_apart(_rand(3, 20, 1, 30), _rand(9, 250, 3, 31)), _apart(_rand(8, 220, 3, 32), _rand(2, 12, 1, 33))]
    return {"one": medium[1:2], "small": small, "medium": medium, "mixed": small + medium + mixed,
            "large": [_rand(11, 330, 3, 41)] + small[:1] + medium[:3] + [_rand(11, 340, 3, 43)]}[kind]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("kind", ["one", "small", "medium", "mixed", "large"])
def test_batches_against_single_runs(kind, dtype):
    import torch
    plans = [jf.plan(i, 1, dtype) for i in _members(kind)]
    want = []
    for p in plans:
        ws = jf.workspace(p.info()["workspace_bytes"])
        want.append(jf.jf_fidelity_alg1(p, ws)["fj"])
        jf.jf_workspace_release(ws)
    ws = jf.workspace(jf.jf_batch_workspace(plans))
    streams = [torch.cuda.Stream(), torch.cuda.default_stream()]
    for rep in range(3):  # replays, with other work between them
        for s in streams:
            for w in (ws, ws[:ws.numel() - 256]):
                print("[gpu-test] batch lanes", kind, dtype, rep, "stream" if s is streams[0] else "null", w.numel(), flush=True)
                try:
                    got = jf.jf_fidelity_batch(plans, w, s)
                except jf.JfError:
                    assert w is not ws and kind in ("one", "small")  # one lane needs as much
                    continue
                assert max(abs(g["fj"] - x) for g, x in zip(got, want)) <= TOL[dtype]
        torch.cuda.synchronize()
        order = list(reversed(range(len(plans))))
        got = jf.jf_fidelity_batch([plans[i] for i in order], ws, streams[0])
        assert max(abs(g["fj"] - want[i]) for g, i in zip(got, order)) <= TOL[dtype]
