"""Batched runs are bitwise those of a run alone, on general stages too: gates
on several qubits, diagonals selected by lanes, quadratic phases, tensor
products formed on load.  Not promised for states that fit one workgroup (13
qubits in complex128, 14 in complex64) whose plan relabels qubits, as a Fourier
transform's SWAPs do: a batch applies their gates one by one."""
import numpy as np
import pytest

from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W
from paper_2604_12256_amd.workloads import Gate

pytestmark = pytest.mark.gpu


def entangled(n, layers, seed):
    """Two-qubit unitaries, CNOTs and controlled phases between rotations."""
    rng = np.random.default_rng(seed)
    gates = []
    for _ in range(layers):
        gates += [Gate("RY", (q,), float(rng.uniform(0, 6))) for q in range(n)]
        perm = [int(q) for q in rng.permutation(n)]
        for a, b, c, d in zip(perm[0::4], perm[1::4], perm[2::4], perm[3::4]):
            gates.append(Gate("CNOT", (a, b)))
            gates.append(Gate("U", (c, d), 0.0, W.haar_unitary(rng, 4)))
            gates.append(Gate("CPHASE", (b, c), float(rng.uniform(0, 6))))
    return gates


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("family", ["qft", "entangled", "rzz", "diag"])
def test_batch_is_bitwise_the_run_alone(family, dtype):
    import torch
    make = {"qft": W.qft, "entangled": lambda n, s: entangled(n, 4, s), "rzz": W.rzz_full,
            "diag": lambda n, s: W.diag_heavy(n, 150, s)}[family]
    sims = []
    for i in range(12):
        n = (15 if family == "qft" else 12) + i % 6
        sims.append(qsim.Simulator(n, dtype=dtype, opt=qsim.OPT_ALL))
        sims[-1].load(make(n, i))
    print(f"batch against alone: {family} {dtype}", flush=True)
    qsim.run_batch(sims)
    torch.cuda.synchronize()
    together = [s.amplitudes() for s in sims]
    differ = []
    for i, s in enumerate(sims):
        s.run()
        if not np.array_equal(s.amplitudes(), together[i]):
            differ.append(i)
        s.close()
    assert not differ, differ
