"""Plans of circuits with diagonals off the unit circle by less than the input
tolerance (1e-10): an operator that takes a diagonal as a phase must not hold
one.  The exported operators, interpreted, against the oracle, relative to the
largest amplitude (the states are not of norm 1)."""
import numpy as np
import pytest

from paper_2604_12256_amd import qsim
from paper_2604_12256_amd.workloads import Gate
from tests.planinterp import run_plan

PLAIN = qsim.OPT_STAGES | qsim.OPT_FUSE | qsim.OPT_QUAD
TOL = 1e-12  # the package's bound in complex128; unequal moduli add up to 1e-9 and more here


def between_rotations(n, wide):
    """One-qubit diagonals of unequal moduli between rotations of their qubit,
    as gates of their own or as members of wider products of diagonals."""
    gates = [Gate("RX", (q,), 0.3 + 0.1 * q) for q in range(n)]
    gates += [Gate("CZ", (q, (q + 1) % n)) for q in range(n)]
    for i in range(30):
        for q in range(n):
            gates.append(Gate("RX", (q,), 0.2 + 0.07 * (q + i)))
        for q in range(n):
            d = np.exp(1j * np.array([0.1 * q, 0.2 * i]))
            gates.append(Gate("DIAG", (q,), 0.0, d * np.array([1 + 9e-11, 1 - 9e-11])))
            if wide and q % 5 == i % 5:
                gates.append(Gate("CZ", (q, (q + 4) % n)))
        for q in range(n):
            gates.append(Gate("RY", (q,), 0.4 + 0.05 * (q + i)))
    return gates


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("opt", [qsim.OPT_ALL, PLAIN, PLAIN | qsim.OPT_DIAG, qsim.OPT_STAGES])
def test_one_qubit_diagonals_between_rotations(oracle_mod, dtype, opt):
    n = 14
    for wide in (False, True):
        gates = between_rotations(n, wide)
        want = oracle_mod.run(n, gates)
        p = qsim.Plan(n, gates, dtype=dtype, opt=opt)
        err = np.max(np.abs(run_plan(p.ops(), n, p.layout()) - want)) / np.max(np.abs(want))
        assert err < TOL, (wide, err)


@pytest.mark.parametrize("n", [16, 18])
def test_couplings_off_the_unit_circle(oracle_mod, n):
    """Layers of all-pairs diagonals where the quadratic-phase operator is the
    cheapest form: it takes those of modulus 1, and only those."""
    for modulus in (1.0, 1 + 9e-11):
        gates = []
        for layer in range(3):
            for a in range(n):
                for b in range(a):
                    d = modulus * np.exp(1j * (0.1 * np.arange(4) * (a + 1) + 0.03 * b + layer))
                    gates.append(Gate("DIAG", (a, b), 0.0, d))
            gates += [Gate("RX", (q,), 0.3 + 0.1 * q) for q in range(n)]
        gates = [Gate("H", (q,)) for q in range(n)] + gates
        want = oracle_mod.run(n, gates)
        p = qsim.Plan(n, gates, opt=qsim.OPT_ALL)
        ops = p.ops()
        quads = sum(bool(k.get("quad")) for o in ops if o["kind"] == "STAGE" for k in o["kernel_ops"])
        assert (quads > 0) == (modulus == 1.0)
        err = np.max(np.abs(run_plan(ops, n, p.layout()) - want)) / np.max(np.abs(want))
        assert err < TOL, err
