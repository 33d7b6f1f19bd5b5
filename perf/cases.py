"""The work a user of this simulator has it do, as measurable cases.

A case is one of these calls, through the package's public entry points:

* solve    -- plan a circuit and run it from |0...0> (`load` + `run`), all
              optimisation passes on.  Up to 14 qubits the whole state is then
              read back (`amplitudes`), as programs at that size do; above,
              the state stays in device memory.
* plain    -- the same with the default options (gate by gate).
* fused    -- the same with gates fused to five qubits on the matrix cores
              (the precision form of the benchmark).
* batch    -- many planned circuits run together (`run_batch`), the request
              server's step.
* energy   -- one evaluation of a QAOA cost: plan and run the circuit for new
              angles, then the expectation of Z_i Z_j for every pair.
* shots    -- plan and run a circuit, then draw shots from the state.
* readout  -- measure a state that is in hand (a saved one, put back into
              the buffer): a marginal, Z strings, a diagonal observable and
              sampled amplitudes.

Sizes are those of the package's workloads, tests and benchmark: 10 to 30
qubits, 10 to 60 layers, complex128 and complex64.
"""
import math
import os
import sys

import numpy as np
import torch

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

from paper_2604_12256_amd import qsim  # noqa: E402
from paper_2604_12256_amd import workloads as W  # noqa: E402

READ_BACK_MAX = 14


def listed():
    return [
        # the smallest request of the serving stream: latency, launches, host planning
        {"name": "solve10_c128", "do": "solve", "family": "layered", "n": 10, "layers": 10, "dtype": "c128"},
        # an ordinary small circuit of odd width, solved and read back whole
        {"name": "solve13_c64", "do": "solve", "family": "layered", "n": 13, "layers": 20, "dtype": "c64"},
        # a server's batch of small requests of mixed widths
        {"name": "batch_small_c128", "do": "batch", "n": 10, "n_max": 13, "layers": 20, "count": 128, "dtype": "c128"},
        # a server's batch of mid-size requests
        {"name": "batch_mid_c128", "do": "batch", "n": 16, "n_max": 16, "layers": 20, "count": 48, "dtype": "c128"},
        # the 22-qubit layered circuit of the parity tests
        {"name": "solve22_c128", "do": "solve", "family": "layered", "n": 22, "layers": 40, "dtype": "c128"},
        # the benchmark's 30-qubit layered circuit, the largest state that most runs use, in both precisions
        {"name": "solve30_c128", "do": "solve", "family": "layered", "n": 30, "layers": 40, "dtype": "c128"},
        {"name": "solve30_c64", "do": "solve", "family": "layered", "n": 30, "layers": 40, "dtype": "c64"},
        # one step of a variational loop: fully-connected QAOA, then all 300 pair correlations
        {"name": "energy25_c128", "do": "energy", "n": 25, "layers": 5, "dtype": "c128"},
        # a Fourier transform, then shots from its result
        {"name": "shots27_c128", "do": "shots", "family": "qft", "n": 27, "layers": 0, "shots": 20000,
         "dtype": "c128"},
        # the outputs of a large state
        {"name": "readout28_c64", "do": "readout", "n": 28, "dtype": "c64"},
        # the default options: one full pass per gate, mostly diagonal gates
        {"name": "plain23_c128", "do": "plain", "family": "diag", "n": 23, "layers": 0, "dtype": "c128"},
        # five-qubit fusion on the matrix cores
        {"name": "fused28_c64", "do": "fused", "family": "layered", "n": 28, "layers": 12, "dtype": "c64"},
    ]


def draw(rng):
    dtype = rng.choice(["c128", "c64"])
    do = rng.choice(["solve", "solve", "solve", "batch", "energy", "shots", "readout", "plain", "fused"])
    if do == "solve":
        family = rng.choice(["layered", "layered", "diag", "qaoa", "rzz"])
        n = rng.randint(10, 30)
        layers = rng.randint(10, 60 if n < 30 else 40) if family == "layered" else rng.randint(1, 5)
        return {"do": do, "family": family, "n": n, "layers": layers, "dtype": dtype}
    if do == "batch":
        n = rng.randint(10, 17)
        count = min(int(round(math.exp(rng.uniform(math.log(3), math.log(128))))), 64 if n > 14 else 128)
        return {"do": do, "n": n, "n_max": min(17, n + rng.randint(0, 3)), "layers": rng.randint(10, 40),
                "count": count, "dtype": dtype}
    if do == "energy":
        return {"do": do, "n": rng.randint(12, 27), "layers": rng.randint(1, 5), "dtype": "c128"}
    if do == "shots":
        # complex128: the drawn basis states depend on the last bits of a complex64 state
        return {"do": do, "family": rng.choice(["qft", "layered"]), "n": rng.randint(11, 28),
                "layers": rng.randint(10, 20), "shots": int(round(math.exp(rng.uniform(math.log(100), math.log(20000))))),
                "dtype": "c128"}
    if do == "readout":
        return {"do": do, "n": rng.randint(16, 29), "dtype": dtype}
    if do == "plain":
        return {"do": do, "family": rng.choice(["diag", "layered"]), "n": rng.randint(12, 25),
                "layers": rng.randint(5, 10), "dtype": dtype}
    return {"do": do, "family": "layered", "n": rng.randint(16, 28), "layers": rng.randint(6, 12), "dtype": dtype}


def _gates(case, seed):
    n, layers, family = case["n"], case["layers"], case["family"]
    if family == "layered":
        return W.layered(n, layers, seed)
    if family == "diag":
        return W.diag_heavy(n, 200, seed)
    if family == "qaoa":
        return W.qaoa_full(n, layers, seed)
    if family == "rzz":
        return W.rzz_full(n, seed)
    if family == "qft":
        return W.qft(n, seed)
    raise ValueError(family)


def _readout_inputs(case, seed):
    rng = np.random.default_rng([seed, 11])
    n = case["n"]
    qubits = [int(q) for q in rng.permutation(n)[:10]]
    masks = [int(m) for m in rng.integers(1, 1 << n, size=24, dtype=np.uint64)]
    on = [int(q) for q in rng.permutation(n)[:6]]
    f = rng.standard_normal(1 << 6)
    idx = rng.integers(0, 1 << n, size=1 << 16, dtype=np.uint64)
    return qubits, masks, on, f, idx


def _saved_state(case, seed):
    """A random state of unit norm, as interleaved (re, im) values."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    real = torch.float64 if case["dtype"] == "c128" else torch.float32
    v = torch.randn(2 << case["n"], dtype=real, device="cuda", generator=g)
    return v.mul_(2.0 ** (-0.5 * (case["n"] + 1)))


def _widths(case):
    """The widths of a batch's circuits: n to n_max in turn."""
    return [case["n"] + i % (case["n_max"] - case["n"] + 1) for i in range(case["count"])]


def _options(case):
    if case["do"] == "plain":
        return {}
    if case["do"] == "fused":
        return {"opt": qsim.OPT_FUSE, "force_fuse_k": 5}
    return {"opt": qsim.OPT_ALL}


def _pairs(n):
    return [(i, j) for i in range(n) for j in range(i + 1, n)]


def prepare(case, seed):
    do, n, dtype = case["do"], case["n"], case["dtype"]
    s = {"do": do, "n": n}
    if do == "batch":
        # one buffer holds every request's state; the server has planned each request as it arrived
        real = torch.float64 if dtype == "c128" else torch.float32
        widths = _widths(case)
        s["states"] = torch.zeros(sum(2 << w for w in widths), dtype=real, device="cuda")
        s["sims"], at = [], 0
        for i, w in enumerate(widths):
            sim = qsim.Simulator(w, dtype=dtype, opt=qsim.OPT_ALL, state=s["states"][at:at + (2 << w)])
            sim.load(W.layered(w, case["layers"], 1000 * seed + i))
            s["sims"].append(sim)
            at += 2 << w
        return s
    s["sim"] = qsim.Simulator(n, dtype=dtype, **_options(case))
    if do == "readout":
        s["in"] = _readout_inputs(case, seed)
        s["sim"].load([W.Gate("H", (q,)) for q in range(n)])
        s["sim"].run()
        s["sim"].state.copy_(_saved_state(case, seed))
        return s
    if do == "energy":
        s["circuit"] = qsim.Circuit(W.qaoa_full(n, case["layers"], seed))
        s["masks"] = [(1 << i) | (1 << j) for i, j in _pairs(n)]
        return s
    s["circuit"] = qsim.Circuit(_gates(case, seed))
    if do == "shots":
        s["u"] = np.random.default_rng([seed, 3]).random(case["shots"])
    return s


def run(s):
    do = s["do"]
    if do == "batch":
        qsim.run_batch(s["sims"])
        return s["states"]
    sim = s["sim"]
    if do == "readout":
        qubits, masks, on, f, idx = s["in"]
        return {"marginal": sim.probabilities(qubits), "z": sim.expect_z(masks), "observable": sim.expect_diagonal(on, f),
                "amplitudes": sim.amplitudes(idx)}
    sim.load(s["circuit"])
    sim.run()
    if do == "energy":
        return {"zz": sim.expect_z(s["masks"])}
    if do == "shots":
        return {"shots": sim.sample(s["u"]).astype(np.int64)}
    if s["n"] <= READ_BACK_MAX:
        return sim.amplitudes().astype(np.complex128 if sim.dtype == "c128" else np.complex64)
    return sim.state


def work(case):
    """The final state written once (or read once, where it is in hand), the
    outputs written, and the arithmetic of the gates at their smallest: a
    diagonal gate on 1 or 2 qubits is one complex multiply per amplitude, a
    one-qubit gate a 2x2 complex product per pair.  With the default options
    each gate is a pass of its own, which reads and writes the state."""
    amp = 16 if case["dtype"] == "c128" else 8
    n, do = case["n"], case["do"]
    if do == "batch":
        layers, widths = case["layers"], _widths(case)
        return {"bytes": sum(amp * 2.0 ** w for w in widths),
                "flops": sum(2.0 ** w * layers * (14.0 * w + 6.0 * (w + w // 4)) for w in widths)}
    amps = 2.0 ** n
    if do == "readout":
        return {"bytes": amp * amps + 8 * (1 << 10) + 8 * 24 + 16 * (1 << 16), "flops": 3.0 * amps}
    if do == "energy":
        pairs = n * (n - 1) // 2
        return {"bytes": amp * amps + 8 * pairs, "flops": amps * case["layers"] * (14.0 * n + 6.0 * pairs)}
    family, layers = case["family"], case["layers"]
    if family == "layered":
        dense, diag = n * layers, layers * (n + n // 4)
    elif family == "diag":
        dense, diag = 40, 160
    elif family == "qaoa":
        dense, diag = n * (layers + 1), layers * n * (n - 1) // 2
    elif family == "rzz":
        dense, diag = n, n * (n - 1) // 2
    else:
        dense, diag = n, n * (n - 1) // 2
    flops = amps * (14.0 * dense + 6.0 * diag)
    if do == "plain":
        return {"bytes": 2.0 * amp * amps * (dense + diag), "flops": flops}
    return {"bytes": amp * amps + 8 * case.get("shots", 0), "flops": flops}


# ---- the same results in plain torch, complex128 ---------------------------

_S2 = math.sqrt(0.5)


def _matrix(g):
    """(is diagonal, entries) of a gate: 2 or 4 diagonal entries, or a 2x2 matrix."""
    k, t = g.kind, g.theta
    e = lambda a: complex(math.cos(a), math.sin(a))  # noqa: E731
    if k == "RZ":
        return True, [e(-t / 2), e(t / 2)]
    if k == "CZ":
        return True, [1, 1, 1, -1]
    if k == "CPHASE":
        return True, [1, 1, 1, e(t)]
    if k == "RZZ":
        return True, [e(-t / 2), e(t / 2), e(t / 2), e(-t / 2)]
    if k == "H":
        return False, [[_S2, _S2], [_S2, -_S2]]
    if k == "X":
        return False, [[0, 1], [1, 0]]
    if k == "SX":
        return False, [[0.5 + 0.5j, 0.5 - 0.5j], [0.5 - 0.5j, 0.5 + 0.5j]]
    if k == "RX":
        c, s = math.cos(t / 2), math.sin(t / 2)
        return False, [[c, -1j * s], [-1j * s, c]]
    if k == "U":
        return False, g.data.tolist()
    raise ValueError(k)


def _simulate(n, gates):
    s = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    s[0] = 1
    for g in gates:
        if g.kind == "SWAP":
            lo, hi = sorted(g.qubits)
            v = s.view(-1, 2, 1 << (hi - lo - 1), 2, 1 << lo)
            t = v[:, 0, :, 1].clone()
            v[:, 0, :, 1] = v[:, 1, :, 0]
            v[:, 1, :, 0] = t
            continue
        diag, m = _matrix(g)
        if len(g.qubits) == 1:
            v = s.view(-1, 2, 1 << g.qubits[0])
            if diag:
                v[:, 0] *= m[0]
                v[:, 1] *= m[1]
            else:
                a, b = v[:, 0], v[:, 1]
                a2 = m[0][0] * a + m[0][1] * b
                b2 = m[1][0] * a + m[1][1] * b
                v[:, 0], v[:, 1] = a2, b2
        else:
            q0, q1 = g.qubits
            lo, hi = min(q0, q1), max(q0, q1)
            v = s.view(-1, 2, 1 << (hi - lo - 1), 2, 1 << lo)
            for b0 in (0, 1):
                for b1 in (0, 1):
                    f = m[b0 + 2 * b1]
                    if f != 1:
                        bl, bh = (b0, b1) if q0 == lo else (b1, b0)
                        v[:, bh, :, bl] *= f
    return s


def _cost(n, gates):
    """Seconds that _simulate takes, roughly."""
    return len(gates) * (6e-5 + 2.0 ** n * 16 * 6 / 3e12)


def _parity_sum(p, mask):
    """sum_x p[x] (-1)^popcount(x & mask)."""
    n = p.numel().bit_length() - 1
    v = p
    for q in range(n - 1, -1, -1):
        v = v.view(2, -1)
        v = v[0] - v[1] if (mask >> q) & 1 else v[0] + v[1]
    return float(v)


def exact(case, seed):
    do, n = case["do"], case["n"]
    if do == "batch":
        if case["count"] * case["layers"] * 2.25 * n > 120000:
            return None
        widths = _widths(case)
        return torch.cat([torch.view_as_real(_simulate(w, W.layered(w, case["layers"], 1000 * seed + i))).reshape(-1)
                          for i, w in enumerate(widths)])
    if do == "energy":
        gates = W.qaoa_full(n, case["layers"], seed)
        if _cost(n, gates) > 12:
            return None
        p = _simulate(n, gates).abs().square()
        return {"zz": np.array([_parity_sum(p, (1 << i) | (1 << j)) for i, j in _pairs(n)])}
    if do == "shots":
        return None
    if do == "readout":
        v = _saved_state(case, seed).to(torch.float64)
        s = torch.view_as_complex(v.view(-1, 2))
        qubits, masks, on, f, idx = _readout_inputs(case, seed)
        p = s.abs().square()

        def marginal(qs):
            keep = sorted(qs)
            v = p.view([2] * n)  # axis a is qubit n - 1 - a
            drop = [n - 1 - q for q in range(n) if q not in qs]
            v = v.sum(dim=drop).reshape(-1).cpu().numpy()  # bit t of the index: keep[t]
            y = np.arange(1 << len(qs))
            at = np.zeros_like(y)
            for t, q in enumerate(qs):
                at |= ((y >> t) & 1) << keep.index(q)
            return v[at]

        return {"marginal": marginal(qubits), "z": np.array([_parity_sum(p, m) for m in masks]),
                "observable": float(marginal(on) @ f),
                "amplitudes": s[torch.from_numpy(idx.astype(np.int64)).cuda()].cpu().numpy()}
    gates = _gates(case, seed)
    if _cost(n, gates) > 12:
        return None
    s = _simulate(n, gates)
    if n <= READ_BACK_MAX:
        return s.cpu().numpy()
    if case["family"] == "qft":
        return None
    return torch.view_as_real(s).reshape(-1)
