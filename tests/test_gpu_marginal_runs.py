"""Marginals over sets with low qubits, where a wave sums runs of 64
amplitudes: fewer than eight runs a segment, eight, several segments, no high
qubit left to sum over.  Against the amplitudes read back; sums of at most
2^16 terms in FP64, 1e-12."""
import numpy as np
import pytest

from oracle import oracle as M
from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [8, 9, 10, 13, 16])
def test_marginal_runs(n, dtype):
    sim = qsim.Simulator(n, dtype=dtype, opt=qsim.OPT_ALL)
    sim.load(W.layered(n, 4, 70 + n))
    sim.run()
    state = sim.amplitudes().astype(np.complex128)
    high = list(range(6, n))
    for qs in ([0], [5], [0] + high, [2] + high[1:], [2] + high[:-1], [1, 4] + high[::2], [3, 0, n - 1], [5] + high[2:]):
        print(f"marginal n={n} {dtype} {qs}", flush=True)
        np.testing.assert_allclose(sim.probabilities(qs), M.marginal(state, qs), rtol=0, atol=1e-12)
    sim.close()
