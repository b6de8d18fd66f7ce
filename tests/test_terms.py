"""Per-tuple traces of Algorithm I, put in tuple order on the device: few of them behind the result,
more in a landing area of their own, many in several chunks, with Kraus counts that are no powers of
two and circuits that fall apart.  Against the emulated program, whose traces the host gathers.
Tolerance 1e-12: both sides compute in complex128."""
import numpy as np
import pytest

from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

CASES = [([3], 1), ([2, 1, 5, 3], 1), ([16, 15], 1), ([1], 1), ([4, 4, 4, 4], 1), ([3, 5, 2, 4], 2), ([2] * 15, 1),
         ([3, 5, 4, 3, 5, 4, 3, 4], 2), ([5, 5, 4, 4, 4, 4, 4, 4], 1), ([3, 2, 2, 3, 1, 4], 3)]


def _inst(counts, parts):
    """Circuits on disjoint qubits, noise places with the given numbers of Kraus operators."""
    rng = np.random.default_rng([len(counts), parts])
    inst = {"n": 0, "gates": [], "noise": []}
    for part in range(parts):
        own = counts[part::parts]
        sub = gen.random_circuit(3, 24, len(own), 0.01, 0.3, 50 + part)
        q0, g0 = inst["n"], len(inst["gates"])
        inst["n"] += sub["n"]
        inst["gates"] += [[g[0], [q + q0 for q in g[1]], g[2]] for g in sub["gates"]]
        for s, nk in zip(sub["noise"], own):
            p = rng.dirichlet(np.ones(nk))
            ops = [np.sqrt(p[k]) * np.linalg.qr(rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)))[0]
                   for k in range(nk)]
            inst["noise"].append({"after": s["after"] + g0, "qubit": s["qubit"] + q0, "kraus": [K.tolist() for K in ops]})
    return inst


@pytest.mark.gpu
@pytest.mark.parametrize("counts,parts", CASES, ids=lambda c: "-".join(map(str, c)) if isinstance(c, list) else str(c))
def test_terms_against_emulation(counts, parts):
    p = jf.plan(_inst(counts, parts), 1, "c128")
    want = p.emulate()
    assert len(want) == int(np.prod(counts))
    ws = jf.workspace(p.info()["workspace_bytes"])
    for k in range(2):  # the landing area is kept by the plan
        print("[gpu-test] terms", counts, parts, "call", k, flush=True)
        got = jf.jf_fidelity_alg1(p, ws, want_terms=True)
        assert got["terms"].dtype == np.complex128 and got["terms"].shape == want.shape
        assert np.max(np.abs(got["terms"] - want)) <= 1e-12
        assert abs(got["fj"] - np.sum(np.abs(want) ** 2)) <= 1e-11
    none = jf.jf_fidelity_alg1(p, ws)
    assert "terms" not in none and none["fj"] == got["fj"]
    free = jf.jf_fidelity_noalloc(p, want_terms=True)
    assert np.max(np.abs(free["terms"] - want)) <= 1e-12
