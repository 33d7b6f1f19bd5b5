"""Plans of stages that run on the rotation kernel (one-qubit gates and
diagonals), checked against the oracle by interpreting their exported
operators: rotations as the shears the kernel applies, tables on all register
bits, lane-selected diagonals.  Which stages take that route is checked too:
the exported tables name every register bit."""
import numpy as np
import pytest

from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W
from paper_2604_12256_amd.workloads import Gate
from tests.planinterp import run_plan


def gate_mix(n, layers, seed):
    """Every one-qubit kind, gates at the edges of the decomposition (exact
    exchanges, equal halves, identities), and diagonals on one to three
    qubits, about one coupling a one-qubit gate."""
    rng = np.random.default_rng(seed)
    kinds = ["H", "X", "Y", "Z", "S", "T", "SX", "RX", "RY", "RZ", "U"]
    angles = [1e-3, np.pi, -np.pi, np.pi / 2, 1e-9, np.pi - 1e-9]
    gates = []
    for _ in range(layers):
        for q in rng.permutation(n):
            k = kinds[int(rng.integers(0, len(kinds)))]
            th = float(angles[int(rng.integers(0, 6))]) if rng.random() < 0.5 else float(rng.uniform(0, 6))
            gates.append(Gate(k, (int(q),), th, W.haar_unitary(rng, 2) if k == "U" else None))
            if rng.random() < 0.7:
                k = 3 if n > 2 and rng.random() < 0.1 else 2
                qs = tuple(int(x) for x in rng.permutation(n)[:k])
                kind = "DIAG" if k == 3 or rng.random() < 0.2 else ("CZ", "CPHASE", "RZZ")[int(rng.integers(0, 3))]
                data = np.exp(1j * rng.uniform(0, 6, 1 << k)) if kind == "DIAG" else None
                gates.append(Gate(kind, qs, float(rng.uniform(0, 6)), data))
    return gates


def rotation_stages(ops, reg):
    n = 0
    for o in ops:
        if o["kind"] == "STAGE" and any(k["diagonal"] and not k.get("quad") and k["n_register"] == reg
                                        for k in o.get("kernel_ops", [])):
            n += all(k["n_register"] in (0, 1, reg) if k["diagonal"] else len(k["qubits"]) == k["n_register"]
                     for k in o["kernel_ops"])
    return n


@pytest.mark.parametrize("dtype,C", [("c128", c) for c in (10, 11, 12, 13)] + [("c64", c) for c in (11, 12, 13, 14)])
def test_rotation_plans_match_the_oracle(oracle_mod, dtype, C):
    reg = 4 if dtype == "c128" else 5
    used = 0
    for n in (C, C + 1, 15):
        for name, gates in (("layered", W.layered(n, 5, C)), ("mix", gate_mix(n, 3, 10 * C + n)),
                            ("product", W.product_circuit(n, 5, n)),
                            ("swaps", W.layered(n, 2, 3) + [Gate("SWAP", (0, n - 1))] + W.layered(n, 2, 4))):
            want = oracle_mod.run(n, gates)
            for opt in (qsim.OPT_ALL, qsim.OPT_STAGES | qsim.OPT_FUSE):
                p = qsim.Plan(n, gates, dtype=dtype, C=C, opt=opt)
                ops = p.ops()
                used += rotation_stages(ops, reg)
                for use_k in (True, False):
                    got = run_plan(ops, n, p.layout(), use_kernel_ops=use_k)
                    assert np.max(np.abs(got - want)) < 1e-12, (name, n, opt, use_k)
    assert used > 10


def test_general_stages_keep_the_general_kernel(oracle_mod):
    """Stages with gates on several qubits, many diagonals a one-qubit gate,
    a matrix only unitary to 1e-11, a dense gate without off-diagonal entries, or
    no fusion."""
    n = 13
    rng = np.random.default_rng(3)
    u = W.haar_unitary(rng, 2)
    u = u + 3e-11 * np.array([[1, 1j], [0.5, 1]])
    cases = [(W.layered(n, 3, 1) + [Gate("CNOT", (3, 9))], qsim.OPT_STAGES | qsim.OPT_FUSE),
             (W.qaoa_full(n, 2, 3), qsim.OPT_STAGES | qsim.OPT_FUSE),
             ([Gate("U", (q,), 0.0, u) for q in range(n)], qsim.OPT_STAGES | qsim.OPT_FUSE),
             (W.layered(n, 3, 1) + [Gate("RX", (3,), 0.0)], qsim.OPT_STAGES | qsim.OPT_FUSE),  # needs no register
             (W.layered(n, 3, 1), qsim.OPT_STAGES)]
    for gates, opt in cases:
        p = qsim.Plan(n, gates, C=13, opt=opt)
        ops = p.ops()
        assert rotation_stages(ops, 4) == 0
        assert np.max(np.abs(run_plan(ops, n, p.layout()) - oracle_mod.run(n, gates))) < 1e-12


def test_offload_passes_with_rotations(oracle_mod):
    n = 16
    for dtype, W_ in (("c128", 12), ("c64", 13)):
        for gates in (W.layered(n, 4, 8), gate_mix(n, 2, 9)):
            p = qsim.Plan(n, gates, dtype=dtype, offload_window=W_)
            assert np.max(np.abs(run_plan(p.ops(), n, p.layout()) - oracle_mod.run(n, gates))) < 1e-12
