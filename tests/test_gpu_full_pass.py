"""Full-pass kernels at their edges, gate by gate against the CPU oracle
(1e-12 in complex128, 2e-5 of the largest amplitude in complex64): diagonals
whose exact ones make qubits controls, at every position around a cache line,
and fused-size dense gates on the smallest states the matrix-core kernel
takes, on low, high and mixed qubits in any order."""
import numpy as np
import pytest

from oracle import oracle
from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W
from paper_2604_12256_amd.workloads import Gate

pytestmark = pytest.mark.gpu


def check(n, gates, dtype, what, **kw):
    print(f"{what} n={n} {dtype}", flush=True)
    sim = qsim.Simulator(n, dtype=dtype, **kw)
    sim.load(gates)
    sim.run()
    got, want = sim.amplitudes(), oracle.run(n, gates)
    sim.close()
    tol = 1e-12 if dtype == "c128" else 2e-5 * float(np.max(np.abs(want)))
    err = float(np.max(np.abs(got - want)))
    assert err <= tol, f"{what} n={n}: {err:.2e} > {tol:.2e}"


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_diagonal_controls(dtype):
    rng = np.random.default_rng(1)
    for n in (1, 2, 3, 4, 5, 6, 9, 12):
        gates = [Gate("U", (q,), 0.0, W.haar_unitary(rng, 2)) for q in range(n)]
        for q in range(n):
            gates += [Gate("Z", (q,)), Gate("T", (q,)), Gate("RZ", (q,), 0.3 + q)]
            for p in range(n):
                if p != q:
                    gates += [Gate("CZ", (q, p)), Gate("CPHASE", (q, p), 0.1 + q + p), Gate("RZZ", (q, p), 0.7)]
        for k in range(1, min(n, 6) + 1):
            for _ in range(6):
                # exact ones everywhere but where some random qubits have random values
                d = np.exp(1j * rng.uniform(0, 6, 1 << k))
                y = np.arange(1 << k)
                ctl, val = int(rng.integers(0, 1 << k)), int(rng.integers(0, 1 << k))
                d[(y & ctl) != (val & ctl)] = 1.0
                gates.append(Gate("DIAG", tuple(int(x) for x in rng.permutation(n)[:k]), 0.0, d))
            gates.append(Gate("DIAG", tuple(int(x) for x in rng.permutation(n)[:k]), 0.0, np.ones(1 << k, complex)))
        check(n, gates, dtype, "controls")


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("k", [3, 4, 5])
def test_matrix_core_smallest_states(k, dtype):
    rng = np.random.default_rng(k)
    for n in (k + 3, k + 4, k + 5, k + 7):
        gates = [Gate("U", (q,), 0.0, W.haar_unitary(rng, 2)) for q in range(n)]
        sets = [range(k), range(n - k, n), reversed(range(k))] + [rng.permutation(n)[:k] for _ in range(4)]
        gates += [Gate("U", tuple(int(x) for x in s), 0.0, W.haar_unitary(rng, 1 << k)) for s in sets]
        check(n, gates, dtype, f"k={k}")
