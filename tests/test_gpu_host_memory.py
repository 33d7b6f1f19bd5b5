"""Host memory that a context keeps between loads: its plan, and buffers of a
few MiB, not the largest load it ever made."""
import ctypes
import resource

import pytest

from paper_2604_12256_amd import qsim
from paper_2604_12256_amd.workloads import Gate

pytestmark = pytest.mark.gpu


def resident():
    ctypes.CDLL(None).malloc_trim(0)
    return int(open("/proc/self/statm").read().split()[1]) * resource.getpagesize()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_a_large_load_is_given_back(dtype):
    n = 20
    layer = [Gate("CPHASE", (a, b), 0.1 + 0.01 * a) for a in range(n) for b in range(a)]
    large = []
    for q in range(3):  # three tables of 2^20 entries
        large += layer + [Gate("H", (q,))]
    small = [Gate("H", (0,))]

    def cycle():
        sim = qsim.Simulator(n, dtype=dtype, opt=qsim.OPT_STAGES | qsim.OPT_DIAG, D=20)
        sim.load(large)
        sim.load(small)
        return sim

    cycle().close()  # the runtime's own buffers are there now
    before = resident()
    sims = [cycle() for _ in range(4)]
    kept = (resident() - before) / len(sims)
    for s in sims:
        s.close()
    print(f"{dtype}: {kept / 2**20:.1f} MiB a context", flush=True)
    assert kept < 8 << 20
