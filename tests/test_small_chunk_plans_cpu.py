"""Plans that are only built and read (no context) take any chunk width: below
one wave of register tiles they hold no rotation stage, and below the register
tile itself they are refused."""
import subprocess
import sys
import textwrap

import pytest

CHILD = """
import numpy as np
from oracle import oracle
from paper_2604_12256_amd import qsim
from paper_2604_12256_amd import workloads as W
from tests.planinterp import run_plan
n, reg = 13, {reg}
for name, gates in (("qaoa", W.qaoa_full(n, 2, 1)), ("layered", W.layered(n, 4, 1)), ("qft", W.qft(n, 1))):
    want = oracle.run(n, gates)
    for C in range(1, reg + 10):
        try:
            p = qsim.Plan(n, gates, dtype="{dtype}", C=C)
        except qsim.QsimError:
            assert C < reg, (name, C)
            continue
        assert C >= reg, (name, C)
        assert np.max(np.abs(run_plan(p.ops(), n, p.layout()) - want)) < 1e-12, (name, C)
print("done")
"""


@pytest.mark.parametrize("dtype,reg", [("c128", 4), ("c64", 5)])
def test_any_chunk_width(oracle_mod, dtype, reg):
    # in a process of its own: a read past a thread map ends the process
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(CHILD.format(dtype=dtype, reg=reg))],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "done" in r.stdout, (r.returncode, r.stderr[-500:])
