"""Rounding of the factors that a plan multiplies the state by, in extended
precision (numpy's long double)."""
import numpy as np
import pytest

from paper_2604_12256_amd import qsim
from paper_2604_12256_amd.workloads import Gate

WIDE = np.clongdouble
U = 2.0 ** -53
TABLES = qsim.OPT_STAGES | qsim.OPT_FUSE


def diagonal(n, qubits, table):
    x = np.arange(1 << n, dtype=np.int64)
    y = np.zeros_like(x)
    for j, q in enumerate(qubits):
        y |= ((x >> q) & 1) << j
    return np.asarray(table, dtype=WIDE)[y]


@pytest.mark.parametrize("opt", [TABLES, TABLES | qsim.OPT_DIAG])
def test_tables_are_rounded_once(opt):
    """A circuit of diagonals: the product of the plan's tables against the
    product of the gates' own entries.  Each table entry is rounded once, to
    within 2^-53 of its modulus 1."""
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no extended precision on this host")
    n = 12
    for seed in range(4):
        rng = np.random.default_rng(seed)
        gates = []
        for rep in range(5):
            gates += [Gate("DIAG", (a, b), 0.0, np.exp(1j * rng.uniform(0, 6, 4))) for a in range(n) for b in range(a)]
            gates += [Gate("DIAG", (q,), 0.0, np.exp(1j * rng.uniform(0, 6, 2))) for q in range(n)]
            gates.append(Gate("DIAG", (1, 7, 4), 0.0, np.exp(1j * rng.uniform(0, 6, 8))))
        want = np.ones(1 << n, dtype=WIDE)
        for g in gates:
            want = want * diagonal(n, g.qubits, g.data)
        p = qsim.Plan(n, gates, opt=opt, C=10)
        got, tables = np.ones(1 << n, dtype=WIDE), 0
        for op in p.ops():
            if op["kind"] == "STAGE":
                for k in op["kernel_ops"]:
                    assert k["diagonal"] and not k.get("quad")
                    got, tables = got * diagonal(n, k["qubits"], k["payload"]), tables + 1
            else:
                assert op["kind"] == "INIT"
        assert 0 < tables < len(gates) / 10
        # a detector's product on up to three qubits is rounded before it joins
        # a table (one that ends such a run, at most)
        rounded = 2 if opt & qsim.OPT_DIAG else 1
        err = float(np.max(np.abs(got / want - 1)))
        assert err <= 1.01 * U * rounded * tables, (seed, err / U, tables)
