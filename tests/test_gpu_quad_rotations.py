"""Rotation stages with quadratic phases against the oracle: smallest, tuned
and largest chunks, one chunk and many, and batches that mix them with other
stages.  1e-12 in complex128, 2e-5 of the largest amplitude in complex64."""
import numpy as np
import pytest

from oracle import oracle
from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W
from tests.test_quad_rotations_cpu import PLAIN, families

pytestmark = pytest.mark.gpu


def check(got, want, dtype, what):
    tol = 1e-12 if dtype == "c128" else 2e-5 * float(np.max(np.abs(want)))
    err = float(np.max(np.abs(got - want)))
    assert err <= tol, f"{what}: {err:.2e} > {tol:.2e}"


@pytest.mark.parametrize("dtype,C", [("c128", c) for c in (10, 12, 13)] + [("c64", c) for c in (11, 13, 14)])
def test_quad_rotations(dtype, C):
    for n in (C, C + 1, 17):
        for name, gates in families(n, n + C):
            want = oracle.run(n, gates)
            for opt in (qsim.OPT_ALL, PLAIN):
                print(f"quad rotations {name} n={n} C={C} {dtype} opt={opt}", flush=True)
                sim = qsim.Simulator(n, dtype=dtype, opt=opt, C=C)
                sim.load(gates)
                sim.run()
                check(sim.amplitudes(), want, dtype, f"{name} n={n} C={C}")
                sim.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_batch(dtype):
    import torch
    cases = []
    for i in range(9):
        n = 14 + i % 3
        gates = (W.qaoa_full(n, 2, i), W.layered(n, 3, i), W.qft(n, i))[i // 3]
        sim = qsim.Simulator(n, dtype=dtype, opt=qsim.OPT_ALL)
        sim.load(gates)
        cases.append((n, gates, sim))
    print(f"quad rotations batch {dtype}", flush=True)
    qsim.run_batch([c[2] for c in cases])
    torch.cuda.synchronize()
    for i, (n, gates, sim) in enumerate(cases):
        got = sim.amplitudes()
        check(got, oracle.run(n, gates), dtype, f"batch {i}")
        if dtype == "c128" or i < 6:  # complex64 general stages round differently in a batch
            sim.run()
            assert np.array_equal(sim.amplitudes(), got), i
        sim.close()
