"""Tiles of zeros, which the register-tile kernel leaves as they are, against the
oracle: states with one amplitude that is not zero at each corner of a tile (first
and last register, lane and wave; first and last tile), of minus zeros, and dense
ones with a few tiles of zeros, through passes that mix, move and multiply by
tables; large coefficients run on zeros too.  About 100 gates
of a few eps each: 1e-12 (complex128), 1e-4 (complex64), norm of the difference."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(0, 0), (11, 3), (12, 3), (13, 4), (13, 5)]


def sparse_states(n, rng):
    for at in (0, 1, 63, 64, 2047, (1 << n) - 1, 5 << (n - 4)):
        psi = np.zeros(1 << n, dtype=np.complex128)
        psi[at] = 1j
        yield psi
    psi = np.full(1 << n, complex(-0.0, -0.0))
    psi[3 << (n - 3)] = 1.0
    yield psi
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi.reshape(16, -1)[rng.permutation(16)[:9]] = 0      # blocks of the highest bits
    psi.reshape(-1, 16)[:, 3] = 0                         # and of the lowest
    yield psi / np.linalg.norm(psi)


def circuit(n, rng):
    c = W.config1_random(n, layers=2)
    for q in range(0, n - 1, 2):
        c.add(W.phase(float(rng.uniform(0, 6))), (q,), (n - 1 - q,) if n - 1 - q != q else (0,))
    c.add(W.haar_2x2(rng), (0,), (n - 1,))
    return c


@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 1e-4)])
@pytest.mark.parametrize("tile_bits,reg_bits", SHAPES)
def test_sparse_states(tile_bits, reg_bits, dtype, tol):
    from paper_1612_08091_amd import qsv
    n = 17
    rng = np.random.default_rng(tile_bits + reg_bits)
    s = qsv.Simulator(n_max=n, mode="tiled", tile_bits=tile_bits, reg_bits=reg_bits, dtype=dtype,
                      use_torch_stream=False)
    s.allocate(n)
    for psi in sparse_states(n, rng):
        circ = circuit(n, rng)
        s.set_state(psi)
        s.run(circ)
        assert np.linalg.norm(s.get_state() - oracle.run(circ, psi.copy())) <= tol
    s.close()


@pytest.mark.parametrize("big", [3.0, 1e200])
def test_large_coefficients(big):
    from paper_1612_08091_amd import qsv
    n = 14
    s = qsv.Simulator(n_max=n, mode="tiled", use_torch_stream=False)
    s.allocate(n)
    u = np.array([[big, 1.0], [0.5, 1.0]])
    s.apply(u.astype(complex), (13,))
    got = s.get_state()
    s.close()
    want = np.zeros(1 << n, dtype=complex)
    want[0] = 1.0
    want = (u @ want.reshape(2, -1)).reshape(-1)
    assert np.max(np.abs(got - want)) <= 1e-14 * big
