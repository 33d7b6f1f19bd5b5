"""The rotation kernel against the oracle: every chunk size (one wave to a
whole workgroup of register tiles), one chunk and many, edge gates of the
decomposition, lane, wave and chunk couplings, tensor products formed on load,
batches mixed with general stages, and offload windows.  1e-12 in complex128,
2e-5 of the largest amplitude in complex64."""
import numpy as np
import pytest

from oracle import oracle
from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W
from tests.test_rotation_stages_cpu import gate_mix

pytestmark = pytest.mark.gpu


def check(got, want, dtype, what):
    tol = 1e-12 if dtype == "c128" else 2e-5 * float(np.max(np.abs(want)))
    err = float(np.max(np.abs(got - want)))
    assert err <= tol, f"{what}: {err:.2e} > {tol:.2e}"


@pytest.mark.parametrize("dtype,C", [("c128", c) for c in (10, 11, 12, 13)] + [("c64", c) for c in (11, 12, 13, 14)])
def test_chunk_sizes(dtype, C):
    for n in (C, C + 1, 17):
        for name, gates in (("layered", W.layered(n, 6, C)), ("mix", gate_mix(n, 3, 10 * C + n))):
            want = oracle.run(n, gates)
            for opt in (qsim.OPT_ALL, qsim.OPT_STAGES | qsim.OPT_FUSE):
                print(f"rotations {name} n={n} C={C} {dtype} opt={opt}", flush=True)
                sim = qsim.Simulator(n, dtype=dtype, opt=opt, C=C)
                sim.load(gates)
                sim.run()
                check(sim.amplitudes(), want, dtype, f"{name} n={n} C={C}")
                sim.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_batch_with_general_stages(dtype):
    import torch
    cases = []
    for i in range(70):
        n = 12 + i % 5
        gates = (W.layered(n, 3, i), W.qaoa_full(n, 1, i), W.random_mixed(n, 60, i, max_k=2))[i % 3]
        sim = qsim.Simulator(n, dtype=dtype, opt=qsim.OPT_ALL)
        sim.load(gates)
        cases.append((n, gates, sim))
    print(f"mixed batch {dtype}", flush=True)
    qsim.run_batch([c[2] for c in cases])
    torch.cuda.synchronize()
    for i, (n, gates, sim) in enumerate(cases):
        if i < 15 or i > 60:
            check(sim.amplitudes(), oracle.run(n, gates), dtype, f"batch {i}")
        sim.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_offload_windows(dtype):
    n = 17
    for gates in (W.layered(n, 4, 8), gate_mix(n, 2, 9)):
        print(f"offload {dtype}", flush=True)
        sim = qsim.Simulator(n, dtype=dtype, opt=qsim.OPT_ALL, offload_window=14)
        sim.load(gates)
        sim.run()
        check(sim.amplitudes(), oracle.run(n, gates), dtype, "offload")
        sim.close()
