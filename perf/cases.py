"""The fidelity work that users of this library have it do, as timed cases.

A case names a circuit family with its sizes, the algorithm, the arithmetic form and how the
program keeps its plan.  The circuit's structure (gates, wires, noise places) comes from the case;
the seed draws the RZ angles and the noise strengths, so every seed is another input of the same
shape.  A pass is one call of a fidelity entry point on a kept plan, workspace and stream."""
import math

import numpy as np
import torch

from paper_2103_11595_amd import instances, jf

# Families: "random" (70% one-qubit gates from {H, S, T, RZ}, 30% CX, depolarising noise), "chain"
# (brickwork of RZ + SX layers and CX, depolarising and amplitude damping alternating), "haar"
# (brickwork of Haar SU(2) layers and CX, depolarising), "batch" (random circuits of uneven sizes up
# to n, gates and sites).  alg 0 lets the planner choose; cap is the size cap in log2 elements (0:
# the default); effort is the planner's search effort (0: its own sizing); graph replays the pass
# as a hipGraph on a stream of its own; tuned runs the kernel autotuner once, as a program that
# keeps its plan does; terms also returns the trace of every Kraus tuple.
_DEFAULTS = {"alg": 1, "dtype": "c64", "cap": 0, "effort": 6, "graph": False, "tuned": False, "terms": False, "members": 1}


def _case(name, family, n, gates, sites, circuit, **more):
    return {"name": name, "family": family, "n": n, "gates": gates, "sites": sites, "circuit": circuit, **_DEFAULTS, **more}


def listed():
    return [
        # the smallest call: a five-qubit circuit checked once per call, its 16 traces read back
        _case("rand5_c128_terms", "random", 5, 50, 2, 1, dtype="c128", effort=0, terms=True),
        # an ordinary small circuit with many noise places, the algorithm left to the planner
        _case("rand7_auto_c128", "random", 7, 112, 6, 912, alg=0, dtype="c128"),
        # many Kraus tuples of a ten-qubit circuit: 65536 traces, all read back
        _case("rand10_m8_c128_terms", "random", 10, 200, 8, 708, dtype="c128", effort=8, terms=True),
        # the 16-qubit benchmark circuit in the three forms, plan kept, tuned and replayed
        _case("rand16_c64", "random", 16, 400, 4, 2, effort=8, graph=True, tuned=True),
        _case("rand16_c128", "random", 16, 400, 4, 2, dtype="c128", effort=8, graph=True, tuned=True),
        _case("rand16_bf16x6", "random", 16, 400, 4, 2, dtype="bf16x6", effort=8, graph=True, tuned=True),
        # the 25-qubit noisy chain as one doubled network, plan kept, tuned and replayed
        _case("chain25_c64", "chain", 25, 20, 30, 3, alg=2, graph=True, tuned=True),
        # a shorter odd chain in double precision, planned and called without tuning
        _case("chain19_c128", "chain", 19, 17, 21, 7, alg=2, dtype="c128"),
        # the 36-qubit shallow chain, which falls apart into several small components
        _case("haar36_c64", "haar", 36, 8, 40, 5, alg=2, effort=0, graph=True, tuned=True),
        # a batch of uneven circuits in one submission
        _case("batch40_c64", "batch", 11, 400, 4, 4, effort=3, graph=True, members=40),
        # a plan over its size cap: Kraus indices sliced, one program walked leaf by leaf
        _case("rand10_sliced_c64_terms", "random", 10, 200, 6, 706, cap=18, terms=True),
        # a large circuit called as planned: intermediates of gigabytes
        _case("rand13_c64_large", "random", 13, 360, 4, 24),
    ]


#: flops of the planned contraction that a drawn case stays under (the largest listed case has more)
_MOST_FLOPS = 2.0e11


def _log_between(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    while True:
        kind = rng.choice(["random", "random", "random", "chain", "haar", "batch"])
        case = _case("", kind, 0, 0, 0, rng.randrange(1 << 20))
        case["dtype"] = rng.choice(["c64", "c128", "c64", "c128", "bf16x6"])
        if kind == "random":
            case.update(n=rng.randint(4, 16), gates=_log_between(rng, 30, 500), sites=rng.randint(2, 7))
            case["alg"] = rng.choice([1, 1, 1, 0])
            case["terms"] = case["alg"] == 1 and rng.random() < 0.5
        elif kind == "batch":
            case.update(n=rng.randint(6, 12), gates=_log_between(rng, 50, 400), sites=rng.randint(2, 4),
                        members=_log_between(rng, 4, 60), graph=True, effort=3)
        else:
            case.update(n=rng.randint(9, 36), gates=rng.randint(8, 20), sites=rng.randint(6, 40), alg=2)
        if kind != "batch":
            case["graph"] = case["tuned"] = rng.random() < 0.5
        del case["name"]
        # a random network's cost spans many orders of magnitude: take those with some contraction
        # to run that stay under the largest listed case
        try:
            flops = work(case)["flops"]
        except jf.JfError:
            continue
        if 1e4 <= flops <= _MOST_FLOPS:
            return case


def _instance(case, seed, member=0):
    circuit = case["circuit"]
    if case["family"] == "batch":
        sizes = np.random.default_rng([circuit, member])
        inst = instances.random_circuit(int(sizes.integers(4, case["n"] + 1)), int(sizes.integers(20, case["gates"] + 1)),
                                        int(sizes.integers(1, case["sites"] + 1)), 1e-3, 1e-2, int(sizes.integers(2**31)))
    elif case["family"] == "random":
        inst = instances.random_circuit(case["n"], case["gates"], case["sites"], 1e-3, 1e-2, circuit)
    else:
        mix = ("depolarizing", "amplitude_damping") if case["family"] == "chain" else ("depolarizing",) * 2
        inst = instances.brickwork_chain(case["n"], case["gates"], "rz_sx" if case["family"] == "chain" else "haar",
                                         [(mix[i % 2], 1e-3) for i in range(case["sites"])], circuit)
    values = np.random.default_rng([seed, member])
    for g in inst["gates"]:
        g[2] = [float(x) for x in values.uniform(0.0, 2.0 * math.pi, len(g[2]))]
    for s in inst["noise"]:
        s["p"] = float(values.uniform(1e-3, 1e-2))
    return inst


def _instances(case, seed):
    return [_instance(case, seed, k) for k in range(case["members"])]


def _plan(case, inst):
    flags = jf.JF_FLAG_EFFORT(case["effort"])
    if case["graph"] and case["members"] == 1:
        flags |= jf.JF_FLAG_GRAPH
    return jf.plan(inst, case["alg"], case["dtype"], max_log2=case["cap"], flags=flags)


def prepare(case, seed):
    plans = [_plan(case, inst) for inst in _instances(case, seed)]
    stream = torch.cuda.Stream() if case["graph"] else torch.cuda.current_stream()
    if case["family"] == "batch":
        need = jf.jf_batch_workspace(plans)
    else:
        need = plans[0].info()["workspace_bytes"]
    ws = jf.workspace(need)
    if case["tuned"]:
        jf.jf_autotune(plans[0], ws, stream)
    return {"case": case, "plans": plans, "ws": ws, "stream": stream}


def _result(case, r):
    """F_J, 1 - F_J and the imaginary residual, and the traces, in the precision of the form."""
    wide = case["dtype"] == "c128"
    out = [np.array([r["fj"], r["one_minus_fj"], r["imag_residual"]], np.float64 if wide else np.float32)]
    if case["terms"]:
        out.append(r["terms"].astype(np.complex128 if wide else np.complex64))
    return out


def run(state):
    case, plans, ws, stream = state["case"], state["plans"], state["ws"], state["stream"]
    if case["family"] == "batch":
        return [_result(case, r)[0] for r in jf.jf_fidelity_batch(plans, ws, stream)]
    if plans[0].alg == 1:
        return _result(case, jf.jf_fidelity_alg1(plans[0], ws, stream, want_terms=case["terms"]))
    return _result(case, jf.jf_fidelity_alg2(plans[0], ws, stream))


def work(case):
    """Bytes: every gate matrix and Kraus operator read, every result written.  Flops: those of the
    contraction order that the planner finds (the least of any order is not known)."""
    read = written = flops = 0
    for inst in _instances(case, 0):
        read += sum(16 * 4 ** len(g[1]) for g in inst["gates"])
        kraus = [4 if s["channel"] == "depolarizing" else 2 for s in inst["noise"]]
        read += 64 * sum(kraus)
        written += 24 + (16 * math.prod(kraus) if case["terms"] else 0)
        flops += _plan(dict(case, effort=min(case["effort"] or 6, 6)), inst).info()["path_flops"]
    return {"bytes": read + written, "flops": flops}


# ---------------------------------------------------------------- dense values in 64 bits ---

_ROOT = math.sqrt(0.5)
_FIXED = {"h": [[_ROOT, _ROOT], [_ROOT, -_ROOT]], "s": [[1, 0], [0, 1j]], "t": [[1, 0], [0, complex(_ROOT, _ROOT)]],
          "sx": [[0.5 + 0.5j, 0.5 - 0.5j], [0.5 - 0.5j, 0.5 + 0.5j]]}


def _matrix(gate):
    if gate[0] == "rz":
        half = gate[2][0] / 2
        return np.diag([complex(math.cos(half), -math.sin(half)), complex(math.cos(half), math.sin(half))])
    return np.array(_FIXED[gate[0]], complex)


def _kraus(site):
    p = site["p"]
    paulis = ([[1, 0], [0, 1]], [[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]])
    return [math.sqrt(1 - p if i == 0 else p / 3) * np.array(m, complex) for i, m in enumerate(paulis)]


def _apply(x, n, m, q):
    """The 2 x 2 matrix m on qubit q of the row index of every operator in x (count, 2^n, 2^n)."""
    v = x.view(x.shape[0], 1 << q, 2, -1)
    out = torch.empty_like(v)
    for i in range(2):
        out[:, :, i] = complex(m[i][0]) * v[:, :, 0] + complex(m[i][1]) * v[:, :, 1]
    return out.view_as(x)


def _apply_cx(x, n, c, t):
    lo, hi = min(c, t), max(c, t)
    v = x.view(x.shape[0], 1 << lo, 2, 1 << (hi - lo - 1), 2, -1).clone()
    if c < t:
        v[:, :, 1] = v[:, :, 1].flip(3)
    else:
        v[:, :, :, :, 1] = v[:, :, :, :, 1].flip(2)
    return v.view_as(x)


def _gate(x, n, gate, adjoint=False):
    if gate[0] == "cx":
        return _apply_cx(x, n, *gate[1])
    m = _matrix(gate)
    return _apply(x, n, m.conj().T if adjoint else m, gate[1][0])


def _traces(inst):
    """tr(U^dagger E_k) / 2^n of every Kraus tuple, the first site most significant: the noisy circuit
    is cut in the middle of its sites, P_b the operators up to the cut, V_a those after it taken
    off U from the left, and the traces are the inner products of the two."""
    n, gates, noise = inst["n"], inst["gates"], inst["noise"]
    device = "cuda" if torch.cuda.is_available() else "cpu"
    eye = torch.eye(1 << n, dtype=torch.complex128, device=device)[None]
    ops = []
    for i, g in enumerate(gates):
        ops.append(g)
        ops += [s for s in noise if s["after"] == i]
    cut = [k for k, op in enumerate(ops) if isinstance(op, dict)][len(noise) // 2]
    p = eye
    for op in ops[:cut]:
        if isinstance(op, dict):
            p = torch.stack([_apply(p, n, k, op["qubit"]) for k in _kraus(op)], 1).flatten(0, 1)
        else:
            p = _gate(p, n, op)
    v = eye
    for g in gates:
        v = _gate(v, n, g)
    for op in reversed(ops[cut:]):
        if isinstance(op, dict):
            v = torch.cat([_apply(v, n, k.conj().T, op["qubit"]) for k in _kraus(op)])
        else:
            v = _gate(v, n, op, adjoint=True)
    v = v.flatten(1).conj().resolve_conj().T
    return (p.flatten(1) @ v).flatten().cpu().numpy() / (1 << n)


def exact(case, seed):
    # dense operators: a chain's 2^40 and more Kraus tuples, or more than 13 qubits, are out of their reach
    if case["family"] not in ("random", "batch"):
        return None
    out = []
    for inst in _instances(case, seed):
        if 16.0 * 4 ** (inst["n"] + (len(inst["noise"]) + 1) // 2) > 2**34:
            out.append(None)
            continue
        t = _traces(inst)
        fj = math.fsum(abs(x) ** 2 for x in t)
        out.append(np.array([fj, 1.0 - fj, 0.0]))
        if case["terms"]:
            out.append(t)
    return out if any(x is not None for x in out) else None
