"""Plans of rotation stages around quadratic phases: diagonals on one and two
qubits wait until a rotation needs them and join one operator, those that no
rotation needs pass to the next stage.  The exported operators, interpreted,
against the oracle; which stages take that route."""
import numpy as np
import pytest

from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W
from paper_2604_12256_amd.workloads import Gate
from tests.planinterp import run_plan

PLAIN = qsim.OPT_STAGES | qsim.OPT_FUSE | qsim.OPT_QUAD


def couplings(n, layers, seed):
    """Rotations on every qubit between layers of many couplings: all pairs
    or three in four, in any order, mixed kinds, some with one-qubit diagonals
    among them; the first and the last layer may be couplings."""
    rng = np.random.default_rng(seed)
    gates = []
    for layer in range(layers):
        pairs = [(a, b) if rng.random() < 0.5 else (b, a) for a in range(n) for b in range(a)]
        for i in rng.permutation(len(pairs)):
            if layer % 2 and rng.random() < 0.25:
                continue
            kind = ("RZZ", "CPHASE", "CZ", "DIAG")[int(rng.integers(0, 4))]
            data = np.exp(1j * rng.uniform(0, 6, 4)) if kind == "DIAG" else None
            gates.append(Gate(kind, pairs[i], float(rng.uniform(-7, 7)), data))
            if rng.random() < 0.1:
                gates.append(Gate("RZ", (int(rng.integers(0, n)),), float(rng.uniform(-7, 7))))
        if layer < layers - 1 or seed % 2:
            gates += [Gate("RX" if rng.random() < 0.7 else "U", (q,), float(rng.uniform(0, 6)), W.haar_unitary(rng, 2))
                      for q in range(n)]
    return [Gate(g.kind, g.qubits, g.theta, g.data if g.kind in ("U", "DIAG") else None) for g in gates]


def families(n, seed):
    return (("qaoa", W.qaoa_full(n, 2, seed)), ("couplings", couplings(n, 3, 2 * seed)),
            ("couplings then rotations", couplings(n, 2, 2 * seed + 1)), ("rzz", W.rzz_full(n, seed)))


def quad_rotation_stages(ops, reg):
    return sum(o["kind"] == "STAGE" and any(k.get("quad") for k in o["kernel_ops"]) and
               any(k["diagonal"] and not k.get("quad") and k["n_register"] == reg for k in o["kernel_ops"])
               for o in ops)


@pytest.mark.parametrize("dtype,C", [("c128", c) for c in (10, 12, 13)] + [("c64", c) for c in (11, 13, 14)])
def test_quad_rotation_plans_match_the_oracle(oracle_mod, dtype, C):
    reg = 4 if dtype == "c128" else 5
    used = 0
    for n in (C, C + 1, 16):
        for name, gates in families(n, n + C):
            want = oracle_mod.run(n, gates)
            for opt in (qsim.OPT_ALL, PLAIN, PLAIN | qsim.OPT_DIAG):
                p = qsim.Plan(n, gates, dtype=dtype, C=C, opt=opt)
                ops = p.ops()
                used += quad_rotation_stages(ops, reg)
                for use_k in (True, False):
                    got = run_plan(ops, n, p.layout(), use_kernel_ops=use_k)
                    assert np.max(np.abs(got - want)) < 1e-12, (name, n, opt, use_k)
    assert used > 10


def test_stages_without_the_operator(oracle_mod):
    """No quadratic phases allowed, a diagonal on three qubits, one that is off
    the unit circle by less than the input tolerance, a controlled gate, a
    rotation between every two couplings, host-memory windows."""
    n = 14
    q = couplings(n, 2, 5)
    data = np.exp(1j * np.arange(8))
    cases = [(q, dict(opt=PLAIN & ~qsim.OPT_QUAD)), (q[:30] + [Gate("DIAG", (1, 12, 3), 0.0, data)] + q[30:], dict(opt=PLAIN)),
             (q[:40] + [Gate("DIAG", (2, 11), 0.0, (1 + 3e-11) * data[:4])] + q[40:], dict(opt=PLAIN)),
             (q + [Gate("CNOT", (3, 9))], dict(opt=PLAIN)), (W.qft(n, 3), dict(opt=PLAIN)),
             (q, dict(opt=PLAIN, offload_window=12))]
    for gates, kw in cases:
        p = qsim.Plan(n, gates, **({"C": 10} | kw))
        ops = p.ops()
        if "offload_window" in kw:
            assert quad_rotation_stages(ops, 4) == 0
        assert np.max(np.abs(run_plan(ops, n, p.layout()) - oracle_mod.run(n, gates))) < 1e-12
