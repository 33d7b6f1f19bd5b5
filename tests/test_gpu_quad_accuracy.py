"""Error of quadratic phases in complex128 against extended precision: an
unweighted all-pairs coupling, where every pair has the same coefficient, so
that a coefficient's rounding error meets an amplitude up to n (n - 1) / 2
times over.

Bound on the 2-norm error: a layer multiplies an amplitude about 2 n times by
rotations, 3 times by tables and 30 times on the way through the operator's
running products, each rounding within about 0.6 u at random (u = 2^-53), so
three layers of 19 qubits come to sqrt(3 * 71) * 0.6 u = 9 u; four times that
is allowed.  Coefficients rounded to doubles are off by 0.3 to 1.7 u (angles of
1 to 4), 43 times over for half the bits set: 70 u after three layers."""
import numpy as np
import pytest

from paper_2604_12256_amd import qsim
from paper_2604_12256_amd.workloads import Gate

pytestmark = pytest.mark.gpu

WIDE = np.clongdouble


def rx(theta):
    c, s = np.cos(theta / 2), np.sin(theta / 2)
    return np.array([[c, -1j * s], [-1j * s, c]])


def reference(n, gammas, betas):
    """The circuit gate by gate in extended precision, on the gates' own
    entries: a layer of equal couplings depends on the number of set bits."""
    ones = np.array([bin(x).count("1") for x in range(1 << 10)], dtype=np.int64)
    x = np.arange(1 << n)
    k = ones[x & 1023] + ones[x >> 10]
    psi = np.full(1 << n, np.sqrt(np.longdouble(2)) ** -n, dtype=WIDE)
    for gamma, beta in zip(gammas, betas):
        d = [WIDE(z) for z in np.exp(1j * gamma * np.array([0, 1]))]
        d = [z / abs(z) for z in d]  # the operator takes phases
        f = np.array([d[0] ** (j * (j - 1) // 2 + (n - j) * (n - j - 1) // 2) * d[1] ** (j * (n - j))
                      for j in range(n + 1)], dtype=WIDE)
        psi = psi * f[k]
        m = rx(beta).astype(WIDE)
        for q in range(n):
            t = psi.reshape(-1, 2, 1 << q)
            a, b = t[:, 0], t[:, 1]
            psi = np.stack([m[0, 0] * a + m[0, 1] * b, m[1, 0] * a + m[1, 1] * b], axis=1).reshape(-1)
    return psi


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_equal_couplings(seed):
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no extended precision on this host")
    n, layers = 19, 3
    rng = np.random.default_rng(seed)
    gammas, betas = rng.uniform(1, 4, layers), rng.uniform(0, np.pi, layers)
    gates = [Gate("H", (q,)) for q in range(n)]
    for gamma, beta in zip(gammas, betas):
        z = np.exp(1j * gamma * np.array([0, 1]))
        gates += [Gate("DIAG", (a, b), 0.0, np.array([z[0], z[1], z[1], z[0]])) for a in range(n) for b in range(a)]
        gates += [Gate("U", (q,), 0.0, rx(beta)) for q in range(n)]
    quads = sum(bool(k.get("quad")) for o in qsim.Plan(n, gates).ops() if o["kind"] == "STAGE"
                for k in o["kernel_ops"])
    assert quads >= layers
    print(f"equal couplings n={n} seed={seed}: {quads} quadratic phases", flush=True)
    sim = qsim.Simulator(n, opt=qsim.OPT_ALL)
    sim.load(gates)
    sim.run()
    got = sim.amplitudes()
    sim.close()
    err = float(np.linalg.norm((got - reference(n, gammas, betas)).astype(np.complex128)))
    print(f"2-norm error {err / 2 ** -53:.1f} u", flush=True)
    assert err <= 36 * 2.0 ** -53, err
