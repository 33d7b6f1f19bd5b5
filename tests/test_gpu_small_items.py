"""Small-state items: whole gate lists and booster sub-states in one
workgroup, records and tables copied to LDS in blocks, starting states read,
created or formed as tensor products; batched runs that share their launches.
Tolerances are the package's: 1e-12 against the oracle in complex128, 2e-5 of
the largest amplitude in complex64."""
import numpy as np
import pytest

from oracle import oracle
from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W

pytestmark = pytest.mark.gpu


def check(got, want, dtype, what):
    tol = 1e-12 if dtype == "c128" else 2e-5 * float(np.max(np.abs(want)))
    err = float(np.max(np.abs(got - want)))
    assert err <= tol, f"{what}: {err:.2e} > {tol:.2e}"


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("opt", [0, qsim.OPT_BOOST | qsim.OPT_STAGES, qsim.OPT_ALL])
def test_whole_lists_and_sub_states(dtype, opt):
    """Every width a workgroup holds; gates on up to six qubits (a six-qubit
    matrix stays in global memory, a five-qubit one fills a block), more gates
    than a block holds, and diagonals wider than a word of qubit bytes."""
    import torch
    top = 13 if dtype == "c128" else 14
    cases = []
    for n in range(1, top + 1):
        gates = W.random_mixed(n, 30, 700 + n, max_k=6) + W.layered(n, 4, 800 + n)
        if n >= 5:  # entanglement-free prefix of more than one block, and a lone wide matrix after it
            gates = W.product_circuit(n, 70, 900 + n)[:260] + gates
        sim = qsim.Simulator(n, dtype=dtype, opt=opt)
        sim.load(gates)
        cases.append((n, sim, oracle.run(n, gates)))
    print(f"batch {dtype} opt {opt}", flush=True)
    qsim.run_batch([c[1] for c in cases])
    torch.cuda.synchronize()
    for n, sim, want in cases:
        check(sim.amplitudes(), want, dtype, f"batch n={n}")
        sim.run()
        check(sim.amplitudes(), want, dtype, f"solo n={n}")
        sim.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_more_items_than_a_launch_holds(dtype):
    """130 contexts of four sub-states each: 520 items, 448 to a launch."""
    import torch
    sims = []
    for i in range(130):
        sim = qsim.Simulator(12 if i else 13, dtype=dtype, opt=qsim.OPT_ALL)
        sim.load(W.layered(sim.n, 3, 40 + i))
        sims.append(sim)
    print(f"520 items {dtype}", flush=True)
    qsim.run_batch(sims)
    torch.cuda.synchronize()
    for i, sim in enumerate(sims):
        if i in (0, 1, 64, 111, 112, 113, 129):
            check(sim.amplitudes(), oracle.run(sim.n, W.layered(sim.n, 3, 40 + i)), dtype, f"circuit {i}")
        sim.close()
