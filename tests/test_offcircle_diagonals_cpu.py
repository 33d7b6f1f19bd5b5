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
