"""Reading a plan when memory runs out: the calls report it, the process lives."""
import subprocess
import sys
import textwrap

CHILD = """
import ctypes, resource
import numpy as np
from paper_2604_12256_amd import qsim
from paper_2604_12256_amd.workloads import Gate
n = 22
gates = [Gate("CPHASE", (a, b), 0.1 + 0.01 * a) for a in range(20) for b in range(a)]
p = qsim.Plan(n, gates, opt=qsim.OPT_STAGES | qsim.OPT_FUSE | qsim.OPT_DIAG, D=20)
lib, g = p._lib, qsim.SimPlanGate()
wide = None
for i in range(lib.sim_plan_num_ops(p._p)):
    j = 0
    while lib.sim_plan_stage_gate(p._p, i, j, ctypes.byref(g), None) == qsim.OK:
        if g.payload_len == 1 << 20:
            wide = (i, j)
        j += 1
assert wide is not None
out = np.ones(1 << 20, dtype=np.complex128)
pages = int(open("/proc/self/statm").read().split()[0])
limit = pages * resource.getpagesize() + (16 << 20)   # the table and its factors take 48 MiB
hard = resource.getrlimit(resource.RLIMIT_AS)[1]
resource.setrlimit(resource.RLIMIT_AS, (limit, hard))
assert lib.sim_plan_stage_gate(p._p, *wide, ctypes.byref(g), None) == qsim.OK and g.payload_len == 1 << 20
assert lib.sim_plan_stage_gate(p._p, *wide, ctypes.byref(g), out.ctypes.data) == 2  # out of memory
resource.setrlimit(resource.RLIMIT_AS, (hard, hard))
assert lib.sim_plan_stage_gate(p._p, *wide, ctypes.byref(g), out.ctypes.data) == qsim.OK
assert np.max(np.abs(np.abs(out) - 1)) < 1e-13
print("done")
"""


def test_stage_gate_out_of_memory():
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(CHILD)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "done" in r.stdout, (r.returncode, r.stderr[-600:])
