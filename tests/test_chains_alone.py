"""GPU tests of the chain kernels on small tensors: steps of such sizes run several to a launch by default, so
the Gauss-form kernels are forced here, under which chains stay chains and every other step has a launch
of its own.  Single operators, FP32 pairs (operators that carry noise) and the split form, against the
dense oracle within the bars of the forms (1e-6)."""
import functools

import numpy as np
import pytest

from oracle import dense
from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

pytestmark = pytest.mark.gpu
QUICK = jf.JF_FLAG_EFFORT(2)
PLAIN = QUICK | jf.JF_FLAG_NO_FUSE | jf.JF_FLAG_NO_CANCEL  # one step per tensor: 2 x 2 and 4 x 4 operators
# circuit (n, gates, sites, p range, seed), algorithm, flags, the modes of its chains: 1 single FP32
# operators, 4 with pairs (complex64), 3 the split form
CASES = [((7, 130, 6, 0.01, 0.3, 5115), 2, QUICK), ((7, 39, 6, 0.01, 0.3, 5303), 1, PLAIN), ((7, 39, 6, 0.01, 0.3, 5303), 2, PLAIN),
         ((8, 60, 2, 0.01, 0.3, 3003), 1, PLAIN), ((4, 136, 3, 0.01, 0.3, 2116), 2, QUICK),
         ((8, 220, 3, 1e-3, 0.2, 22), 1, QUICK)]


@functools.lru_cache(None)
def _reference(args):
    ref = dense.fidelity_alg1(gen.random_circuit(*args), want_terms=True)
    return ref["fj"], np.array([ref["terms"][k] for k in sorted(ref["terms"])])


@pytest.mark.parametrize("dtype", ["c64", "bf16x6"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, (c[0][0], c[0][1], c[0][5], c[1], c[2] & 3))))
def test_chains_of_small_tensors(case, dtype):
    args, alg, flags = case
    inst = gen.random_circuit(*args)
    p = jf.plan(inst, alg, dtype, flags=flags)
    if not any(s["chain"] >= 0 for s in p.describe()):
        pytest.skip("no chain in this form")
    fj, terms = _reference(args)
    ws = jf.workspace(p.info()["workspace_bytes"])
    for variant in ("gauss256", "gauss512"):
        jf.jf_set_kernel_variant(p, variant)
        ws.fill_(255)  # NaN wherever a launch leaves something unwritten
        jf.jf_workspace_release(ws)
        print("[gpu-test] chains alone", case, dtype, variant, flush=True)
        got = jf.jf_fidelity_alg1(p, ws, want_terms=True) if alg == 1 else jf.jf_fidelity_alg2(p, ws)
        assert p.last_pass()["grid_launches"] == 0
        assert abs(got["fj"] - fj) <= 1e-6
        if alg == 1:
            assert np.max(np.abs(got["terms"] - terms)) <= 1e-6
        chains = [r for r in jf.jf_profile_steps(p, ws) if r["variant"] == jf.KV_CHAIN]
        assert chains and all(r["steps"] >= 2 for r in chains)
