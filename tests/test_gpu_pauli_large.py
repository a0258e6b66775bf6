"""Coefficients next to the largest double: the sum is finite where each string's
share is.  Rotations on every qubit, so that <X...X> is a product of sines; strings
whose pairs lie in a thread's registers, in lanes, in LDS and in no tile at all, and
the same in the batched form.  Bound: the string's value to 1e-12 (a product of
unitaries and a sum of 2^n products in double; complex64 states 1e-5)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

BIG = 1.5e308
SIN = 0.98


def tilted(n):
    c = W.Circuit(n)
    for q in range(n):
        c.add(W.ry(float(np.arcsin(SIN))), (q,))
    return c


@pytest.mark.parametrize("n", [3, 12, 14, 17])
def test_sum(n):
    from paper_1612_08091_amd import qsv
    s = qsv.Simulator(n_max=n, use_torch_stream=False)
    s.allocate(n)
    s.run(tilted(n))
    for x in (1, 1 << (n - 1), 1 | 1 << (n // 2), (1 << n) - 1):
        want = SIN ** bin(x).count("1")
        assert abs(s.get_expectation([x], [0], [BIG]) / BIG - want) <= 1e-12
        # two strings on one mask whose shares cancel in part
        got = s.get_expectation([x, x, 0], [0, 0, 0], [BIG, -0.9 * BIG, 1.0])
        assert abs(got / BIG - 0.1 * want) <= 1e-12
    s.close()


@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 1e-5)])
def test_batch(dtype, tol):
    from paper_1612_08091_amd import qsv
    n = 14
    xs = [1, 1 << 9, 1 << (n - 1), 1 << (n - 1) | 1 << 8 | 2]
    hams = [W.PauliSum(np.array([x], np.uint64), np.array([0], np.uint64), np.array([BIG])) for x in xs]
    b = qsv.Batch([tilted(n)] * len(xs), hams, dtype=dtype, autotune=False)
    got = b.run() / BIG
    b.close()
    want = np.array([SIN ** bin(x).count("1") for x in xs])
    assert np.max(np.abs(got - want)) <= tol
