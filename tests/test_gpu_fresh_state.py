"""Circuits on a state that begins as |0...0>, of which a pass visits the tiles that
its gates so far can reach: against the same circuit on the same state set from the
host (every tile), bit for bit, and against the oracle.  Sizes from one tile to 2^7
of them; gates on the high qubits first, a large coefficient in the middle (its
zeros are worked on), a second flush.  About 150 gates of a few eps each: 1e-12
(complex128), 1e-4 (complex64), norm of the difference."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(0, 0), (11, 3), (13, 4), (13, 5)]


def circuits(n, rng):
    c = W.config1_random(n, layers=2)
    yield c
    c = W.config1_random(n, layers=1)
    c.gates.reverse()
    for q in range(n - 1, 0, -2):
        c.add(W.haar_2x2(rng), (q,), (n - 1 - q,) if n - 1 - q != q else (0,))
    yield c
    c = W.config1_random(n, layers=1)
    c.gates = c.gates[:3]
    for q in (n - 1, 0, n // 2):
        c.add(W.haar_2x2(rng), (q,))
    yield c


@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 1e-4)])
@pytest.mark.parametrize("tile_bits,reg_bits", SHAPES)
@pytest.mark.parametrize("n", [4, 12, 13, 16, 18])
def test_fresh_state(n, tile_bits, reg_bits, dtype, tol):
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(n + tile_bits + reg_bits)
    for circ in circuits(n, rng):
        states = []
        for fresh in (True, False):
            s = qsv.Simulator(n_max=n, mode="tiled", tile_bits=tile_bits, reg_bits=reg_bits,
                              dtype=dtype, use_torch_stream=False)
            s.allocate(n)
            if not fresh:
                zero = np.zeros(1 << n, dtype=np.complex128)
                zero[0] = 1.0
                s.set_state(zero)
            s.run(circ)
            s.flush()
            first = s.get_state().copy()
            s.run(circ)
            states.append((first, s.get_state().copy()))
            s.close()
        zero = np.zeros(1 << n, dtype=np.complex128)
        zero[0] = 1.0
        once = oracle.run(circ, zero)
        twice = oracle.run(circ, once.copy())
        for a, b, want in zip(*states, (once, twice)):
            assert np.array_equal(a, b)
            assert np.linalg.norm(a - want) <= tol


def test_large_coefficient_between():
    from paper_1612_08091_amd import qsv
    n = 16
    rng = np.random.default_rng(1)
    s = qsv.Simulator(n_max=n, mode="tiled", use_torch_stream=False)
    s.allocate(n)
    want = np.zeros(1 << n, dtype=complex)
    want[0] = 1.0
    gates = [(W.haar_2x2(rng), q) for q in (15, 2, 9)]
    gates.append((np.array([[3.0, 1.0], [0.5, 1.0]], dtype=complex), 14))
    gates += [(W.haar_2x2(rng), q) for q in (0, 13, 1, 12, 11, 3, 15)]
    for u, q in gates:
        s.apply(u, (q,))
        v = want.reshape(-1, 2, 1 << q)
        want = np.einsum("ab,xby->xay", u, v).reshape(-1)
    got = s.get_state()
    s.close()
    assert np.linalg.norm(got - want) <= 1e-12
