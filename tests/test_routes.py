"""GPU tests that passes run as the library says: small steps in launches of their own kind, slices and the
members of a batch in lanes beside each other, and neither where it is switched off or cannot be.
Results against the dense oracle or the emulated program within the bars of the forms (complex128 1e-12,
complex64 1e-6)."""
import numpy as np
import pytest

from oracle import dense
from paper_2103_11595_amd import instances as gen
from paper_2103_11595_amd import jf

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 1e-6}
QUICK = jf.JF_FLAG_EFFORT(1)  # little path search


def _inst(seed):
    return gen.random_circuit(8, 220, 3, 1e-3, 0.2, seed)


def _same(p, got, fj, dtype, reruns=0):
    assert abs(got["fj"] - fj) <= TOL[dtype] and p.last_pass()["reruns"] == reruns


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_small_steps_run_several_to_a_launch(dtype):
    import torch
    inst = _inst(22)
    fj = dense.fidelity_alg1(inst)["fj"]
    side = torch.cuda.Stream()
    p = jf.plan(inst, 1, dtype, flags=QUICK)
    print("[gpu-test] routes of small steps", dtype, flush=True)
    _same(p, jf.jf_fidelity_alg1(p), fj, dtype)
    runs = p.last_pass()["grid_launches"]
    assert runs > 0
    _same(p, jf.jf_fidelity_noalloc(p), fj, dtype)
    assert p.last_pass()["grid_launches"] == runs
    ws = jf.workspace(jf.jf_batch_workspace([p]))
    for stream in (side, None):
        _same(p, jf.jf_fidelity_batch([p], ws, stream)[0], fj, dtype)
        assert p.last_pass()["grid_launches"] == runs
    g = jf.plan(inst, 1, dtype, flags=QUICK | jf.JF_FLAG_GRAPH)
    ws = jf.workspace(g.info()["workspace_bytes"])
    for _ in range(2):
        _same(g, jf.jf_fidelity_alg1(g, ws, side), fj, dtype)
        assert g.last_pass()["grid_launches"] == runs
    q = jf.plan(inst, 1, dtype, flags=QUICK | jf.JF_FLAG_NO_CHAIN)
    _same(q, jf.jf_fidelity_alg1(q), fj, dtype)
    assert q.last_pass()["grid_launches"] == 0
    jf.jf_set_kernel_variant(p, jf.KV_FMA)
    _same(p, jf.jf_fidelity_alg1(p), fj, dtype)
    assert p.last_pass()["grid_launches"] == 0
    jf.jf_set_kernel_variant(p, jf.KV_AUTO)
    _same(p, jf.jf_fidelity_alg1(p), fj, dtype)
    assert p.last_pass()["grid_launches"] == runs


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_slices_and_members_run_in_lanes(dtype):
    import torch
    inst = gen.random_circuit(8, 220, 6, 0.01, 0.3, 21)
    cap = int(jf.plan(inst, 1, dtype, flags=QUICK).info()["max_log2_intermediate"]) - 2
    p = jf.plan(inst, 1, dtype, max_log2=cap, flags=QUICK)
    assert p.stats()["n_sliced_sites"] > 0 and p.stats()["n_sliced_wires"] == 0
    want = np.sum(np.abs(p.emulate()) ** 2)
    size = p.info()["workspace_bytes"]
    ws = jf.workspace(size)
    print("[gpu-test] routes of slices", dtype, flush=True)
    for w, lanes in ((ws, 4), (ws[:size - 256], 1)):  # four Kraus operators a site
        _same(p, jf.jf_fidelity_alg1(p, w), want, dtype)
        assert p.last_pass()["lanes"] == lanes
    assert jf.lib().jf_set_grid_wait(p.ptr, 0) == 0  # every lane's barriers give up
    _same(p, jf.jf_fidelity_alg1(p, ws), want, dtype, reruns=1)
    plans = [jf.plan(_inst(seed), 1, dtype, flags=QUICK) for seed in (20, 22, 23)]
    fj = [jf.jf_fidelity_alg1(q)["fj"] for q in plans]
    ws = jf.workspace(jf.jf_batch_workspace(plans))
    for stream in (torch.cuda.Stream(), None):
        print("[gpu-test] routes of a batch", dtype, flush=True)
        for q, f, r in zip(plans, fj, jf.jf_fidelity_batch(plans, ws, stream)):
            _same(q, r, f, dtype)
            assert q.last_pass()["lanes"] > 1 and q.last_pass()["grid_launches"] > 0


@pytest.mark.parametrize("gates, runs", [(600, (20, 40)), (2400, (60, 80))])
def test_long_programs_keep_their_runs_of_small_steps(gates, runs):
    """Programs of 1200 and of 4800 small steps: all of them in runs of up to 48, and as many as the tables
    have room for (3600)."""
    inst = gen.random_circuit(6, gates, 2, 1e-3, 0.2, 18)
    ref = dense.fidelity_alg1(inst, want_terms=True)
    terms = np.array([ref["terms"][k] for k in sorted(ref["terms"])])
    p = jf.plan(inst, 1, "c128", flags=QUICK | jf.JF_FLAG_NO_FUSE | jf.JF_FLAG_NO_CANCEL)
    assert p.stats()["n_steps"] >= 2 * gates
    for run in (jf.jf_fidelity_alg1, jf.jf_fidelity_noalloc):
        print("[gpu-test] a long program", gates, run.__name__, flush=True)
        got = run(p, want_terms=True)
        assert np.max(np.abs(got["terms"] - terms)) <= 1e-12 and p.last_pass()["reruns"] == 0
        assert runs[0] <= p.last_pass()["grid_launches"] <= runs[1]


@pytest.mark.parametrize("dtype", ["c128"])  # tensors of 2^16 elements, tiles of 2^12 at most
def test_blocks_of_other_tiles_are_timed_apart(dtype):
    """Tuning: blocks of the same step sizes whose legs lie elsewhere are other launches."""
    inst = gen.random_circuit(8, 500, 2, 1e-3, 0.2, 19)
    fj = dense.fidelity_alg1(inst)["fj"]
    flags = QUICK | jf.JF_FLAG_NO_FUSE | jf.JF_FLAG_NO_CANCEL | jf.JF_FLAG_SMALL_BLOCKS
    p = jf.plan(inst, 1, dtype, flags=flags)
    ws = jf.workspace(p.info()["workspace_bytes"])
    steps, sizes, at = p.describe(), set(), 0
    for launch in jf.jf_profile_steps(p, ws):
        own = steps[at:at + launch["steps"]]
        at += launch["steps"]
        if launch["variant"] == jf.KV_BLOCK:
            sizes.add(tuple((s["kS"], s["kN"], s["rA"], s["rC"], s["chain"] >= 0) for s in own))
    assert at == len(steps)
    print("[gpu-test] tuning blocks", dtype, "sizes", len(sizes), flush=True)
    jf.jf_autotune(p, ws, reps=1)
    timed = p.last_pass()["joint_timings"]
    assert timed > len(sizes) > 0
    jf.jf_autotune(p, ws, reps=1)
    assert p.last_pass()["joint_timings"] == 0  # known by now
    _same(p, jf.jf_fidelity_alg1(p, ws), fj, dtype)
