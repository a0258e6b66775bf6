"""Pinned host blocks of a handle (each costs microseconds to allocate and to free):
one for a flush and the reductions after it, none before there is something to
upload or to read, and results that outlive an upload slot that has grown.  The
library logs its blocks under QSV_LOG=2, read at its first use: a child process."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CHILD = """
import sys
import numpy as np
import workloads as W
from paper_1612_08091_amd import qsv

def mark(name):
    print("--", name, file=sys.stderr, flush=True)

n = 6
s = qsv.Simulator(n_max=n, use_torch_stream=False)
s.allocate(n)
mark("state")
s.synchronize()
s.state_pointer()
mark("flush and reductions")
s.apply(W.H, [0])
s.flush()
assert abs(s.get_probability([0], [1]) - 0.5) < 1e-12
assert s.sample([0.25, 0.75]).tolist() == [0, 1]
assert s.measure([0], [0.75]) == [1]
s.close()
mark("reduction of a state that was set")
s = qsv.Simulator(n_max=n, use_torch_stream=False)
s.allocate(n)
s.set_state(np.eye(1, 1 << n)[0])
assert s.get_probability([0], [0]) == 1.0
assert s.get_probability([0], [1]) == 0.0
mark("growing uploads")
rng = np.random.default_rng(1)
for terms in (10, 40000, 10, 90000, 90000):
    x = np.zeros(terms, np.uint64)
    z = rng.integers(0, 1 << n, terms).astype(np.uint64)
    assert abs(s.get_expectation(x, z, np.ones(terms)) - terms) < 1e-9 * terms
    assert s.sample([0.5]).tolist() == [0]
s.close()
mark("end")
"""


def test_blocks():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=root, env=dict(os.environ, QSV_LOG="2"),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-4000:]
    blocks, name = {}, ""
    for line in r.stderr.splitlines():
        if line.startswith("-- "):
            name = line[3:]
            blocks[name] = 0
        elif "pinned block" in line:
            blocks[name] += 1
    assert blocks["state"] == 0
    assert blocks["flush and reductions"] == 1
    assert blocks["reduction of a state that was set"] == 1
    assert 4 <= blocks["growing uploads"] <= 5
