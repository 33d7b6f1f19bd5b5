"""Sampling and Z strings at the edges of their kernels: widths around a bin,
a row and a tile; every kind of qubit layout; states with empty bins; more
masks than a launch takes.  Checked against the CPU measurement oracle on the
amplitudes read back, or closed forms; Z strings to 1e-12."""
import numpy as np
import pytest

from oracle import measure as M
from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W
from paper_2604_12256_amd.workloads import Gate

pytestmark = pytest.mark.gpu

LAYOUTS = {"identity": lambda n: [],
           "reversed": lambda n: [(q, n - 1 - q) for q in range(n // 2)],   # every lane bit selects
           "one": lambda n: [(0, n - 1)],                                    # one lane bit selects
           "top": lambda n: [(n - 2, n - 1)],                                # runs, bins out of order
           "mixed": lambda n: [(1, n - 1), (4, n // 2)]}


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("layout", sorted(LAYOUTS))
def test_sample_layouts(layout, dtype):
    rng = np.random.default_rng(3)
    for n in (2, 5, 6, 7, 9, 10, 13, 18, 19):
        swaps = [Gate("SWAP", p) for p in LAYOUTS[layout](n) if 0 <= min(p) and max(p) < n and p[0] != p[1]]
        # entangled on the low and the top qubits only: the X'd qubits in
        # between leave most bins empty
        gates = [g for g in W.layered(n, 3, 50 + n) if all(q < 3 or q >= n - 3 for q in g.qubits)]
        gates += [Gate("X", (q,)) for q in range(3, n - 3) if q % 2] + swaps
        sim = qsim.Simulator(n, dtype=dtype, opt=qsim.OPT_ALL)
        sim.load(gates)
        sim.run()
        state = sim.amplitudes().astype(np.complex128)
        print(f"sample n={n} {layout} {dtype}", flush=True)
        u = rng.random(3000)
        got = sim.sample(u).astype(np.int64)
        cdf = M.cdf(state)
        p = np.abs(state) ** 2
        t = u * cdf[-1]
        assert np.all(p[got] > 0)
        assert np.all(cdf[got] > t - 1e-12) and np.all(np.where(got > 0, cdf[np.maximum(got - 1, 0)], 0.0) <= t + 1e-12)
        assert np.all(np.abs(got - M.sample(state, u).astype(np.int64))[np.minimum(np.abs(cdf[got] - t), np.abs(cdf[got] - p[got] - t)) > 1e-12] == 0)
        sim.close()


@pytest.mark.parametrize("layout", sorted(LAYOUTS))
def test_sample_wide_bins(layout):
    """29 qubits: bins of 128 amplitudes, two strips a shot (uniform state)."""
    n = 29
    sim = qsim.Simulator(n, dtype="c64", opt=qsim.OPT_ALL)
    sim.load([Gate("H", (q,)) for q in range(n)] + [Gate("SWAP", p) for p in LAYOUTS[layout](n)])
    sim.run()
    print(f"sample n={n} {layout}", flush=True)
    k = np.random.default_rng(4).integers(0, 1 << n, size=20000, dtype=np.uint64)
    k[:4] = [0, 1, (1 << n) - 1, 64]
    np.testing.assert_array_equal(sim.sample((k.astype(np.float64) + 0.5) / float(1 << n)), k)
    sim.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_many_z_strings(dtype):
    """Widths below, at and above a tile of 2^12; 1 to 900 masks; a layout
    that moves low qubits to the top."""
    rng = np.random.default_rng(6)
    for n in (1, 2, 6, 11, 12, 13, 16):
        gates = W.layered(n, 3, 90 + n) + ([Gate("SWAP", (0, n - 1)), Gate("SWAP", (1, n - 2))] if n > 5 else [])
        sim = qsim.Simulator(n, dtype=dtype, opt=qsim.OPT_ALL)
        sim.load(gates)
        sim.run()
        state = sim.amplitudes().astype(np.complex128)
        for count in (1, 255, 257, 448, 449, 900):
            masks = [int(m) for m in rng.integers(0, 1 << n, count)]
            print(f"expect_z n={n} {count} {dtype}", flush=True)
            np.testing.assert_allclose(sim.expect_z(masks), M.expect_z(state, masks), rtol=0, atol=1e-12)
        sim.close()
