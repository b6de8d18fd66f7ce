"""Blocks: consecutive steps, size-changing ones among them, applied to one LDS tile.  With
JF_FLAG_SMALL_BLOCKS plans form them at any size, so that small circuits reach every operator shape
(fused: up to 16 x 64 and 64 x 16; one step per tensor: 2 x 2 to 4 x 4, few rows) and the dense oracle
can check them: the tables on the CPU (emulation), the kernel on the GPU.  Tolerances: complex128
1e-12, complex64 1e-6 (the bars of their forms)."""
import sys

import numpy as np
import pytest

from oracle import dense
from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

TOL = {"c128": 1e-12, "c64": 1e-6}
PLAIN = jf.JF_FLAG_NO_FUSE | jf.JF_FLAG_NO_CANCEL
CASES = [(5, 60, 2, 31, 0, 0), (6, 90, 3, 13, 0, 0), (7, 120, 3, 14, 0, 0), (8, 160, 3, 15, 0, 0), (9, 250, 3, 505, 0, 0),
         (6, 70, 4, 15, PLAIN, 0), (8, 60, 2, 3003, PLAIN, 0), (7, 39, 6, 5303, PLAIN, 0), (6, 90, 4, 4242, 0, 2)]


def _inst(case):
    return gen.random_circuit(case[0], case[1], case[2], 0.01, 0.3, case[3])


def _plan(case, dtype, alg=1, flags=0):
    n, gates, sites, seed, fl, cut = case
    inst = _inst(case)
    cap = int(jf.plan(inst, alg, dtype, flags=fl).info()["max_log2_intermediate"]) - cut if cut else 0
    return jf.plan(inst, alg, dtype, max_log2=cap, flags=fl | flags)


def _terms(ref):
    return np.array([ref["terms"][k] for k in sorted(ref["terms"])])


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("case", CASES[:4] + CASES[5:6] + CASES[8:], ids=lambda c: "-".join(map(str, c)))
def test_block_tables_emulated_against_oracle(case, dtype):
    ref = _terms(dense.fidelity_alg1(_inst(case), want_terms=True))
    assert np.max(np.abs(_plan(case, dtype, flags=jf.JF_FLAG_SMALL_BLOCKS).emulate() - ref)) < 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_blocks_against_oracle(case, dtype):
    ref = dense.fidelity_alg1(_inst(case), want_terms=True)
    for alg in (1, 2) if not case[5] else (1,):
        p = _plan(case, dtype, alg, jf.JF_FLAG_SMALL_BLOCKS)
        ws = jf.workspace(p.info()["workspace_bytes"])
        ws.fill_(255)  # NaN wherever a launch leaves something unwritten
        jf.jf_workspace_release(ws)
        print("[gpu-test] blocks", case, "alg", alg, dtype, "steps", p.stats()["n_steps"], flush=True)
        run = jf.jf_fidelity_alg1 if alg == 1 else jf.jf_fidelity_alg2
        kw = {"want_terms": True} if alg == 1 else {}
        got = run(p, ws, **kw)
        assert abs(got["fj"] - ref["fj"]) <= TOL[dtype]
        if alg == 1:
            assert np.max(np.abs(got["terms"] - _terms(ref))) <= TOL[dtype]
        prof = jf.jf_profile_steps(p, ws)
        blocks = [r for r in prof if r["variant"] == jf.KV_BLOCK]
        print("[gpu-test]   launches", len(prof), "blocks of", [r["steps"] for r in blocks], flush=True)
        if p.stats()["n_steps"] >= 12:
            assert blocks
        jf.jf_autotune(p, ws, reps=2)  # blocks kept or split by measurement: same bar
        assert abs(run(p, ws)["fj"] - ref["fj"]) <= TOL[dtype]
        jf.jf_set_kernel_variant(p, "fma")  # every step on its own
        assert not any(r["variant"] == jf.KV_BLOCK for r in jf.jf_profile_steps(p, ws))
        jf.jf_set_kernel_variant(p, "auto")
        assert run(p, ws)["fj"] == got["fj"]
    sys.stdout.flush()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_blocks_of_a_large_plan_against_a_launch_per_step(dtype):
    # 2^24-element intermediates: blocks under the default rule, many tiles a workgroup
    inst = gen.random_circuit(12, 350, 4, 1e-3, 1e-2, 7)
    f = []
    for flags in (0, jf.JF_FLAG_NO_CHAIN):
        p = jf.plan(inst, 1, dtype, flags=jf.JF_FLAG_EFFORT(6) | flags)
        assert p.info()["max_log2_intermediate"] >= 22
        ws = jf.workspace(p.info()["workspace_bytes"])
        f.append(jf.jf_fidelity_alg1(p, ws, want_terms=True))
        if not flags:
            assert any(r["variant"] == jf.KV_BLOCK for r in jf.jf_profile_steps(p, ws))
    assert abs(f[0]["fj"] - f[1]["fj"]) <= TOL[dtype]
    assert np.max(np.abs(f[0]["terms"] - f[1]["terms"])) <= TOL[dtype]
