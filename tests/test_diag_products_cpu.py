"""Tables of products of diagonals on one to six qubits: the plan's tables
against the gates' own entries in extended precision, rounded once each."""
import numpy as np
import pytest

from paper_2604_12256_amd import qsim
from paper_2604_12256_amd.workloads import Gate
from tests.test_factor_accuracy_cpu import U, WIDE, diagonal


@pytest.mark.parametrize("dtype,C", [("c128", 10), ("c128", 12), ("c64", 11)])
def test_products_of_wide_diagonals(dtype, C):
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no extended precision on this host")
    n = 12
    for seed in range(12):
        rng = np.random.default_rng(seed)
        gates = []
        for _ in range(int(rng.integers(1, 40))):
            k = int(rng.integers(1, 7))
            d = np.exp(1j * rng.uniform(0, 6, 1 << k))
            if rng.random() < 0.5:  # controlled phases: most entries exactly 1
                d[rng.random(1 << k) < 0.7] = 1
            gates.append(Gate("DIAG", tuple(int(q) for q in rng.permutation(n)[:k]), 0.0, d))
        want = np.ones(1 << n, dtype=WIDE)
        for g in gates:
            want = want * diagonal(n, g.qubits, g.data)
        got, tables = np.ones(1 << n, dtype=WIDE), 0
        for op in qsim.Plan(n, gates, dtype=dtype, opt=qsim.OPT_STAGES | qsim.OPT_FUSE, C=C).ops():
            for k in op.get("kernel_ops", []):
                got, tables = got * diagonal(n, k["qubits"], k["payload"]), tables + 1
        assert tables > 0
        assert float(np.max(np.abs(got / want - 1))) <= 1.01 * U * tables, (seed, tables)
