"""Sampling against the oracle at the edges of its levels: one block (the
single-kernel path, states below a block and of exactly one), several blocks of
one chunk, several chunks; sparse states whose blocks are mostly zero, a single
amplitude; few shots (through pinned memory) and many.  A shot may differ from
the oracle's only where u T lies within 1e-10 T of the boundary between the two
indices, where either is right, and never takes a zero amplitude."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def state(kind, n, rng):
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    if kind == "sparse":
        psi[rng.random(1 << n) < 1 - 24 / (1 << n)] = 0
        psi[rng.integers(0, 1 << n)] = 1
    elif kind == "one":
        psi[:] = 0
        psi[rng.integers(0, 1 << n)] = 0.5j
    elif kind == "ends":
        psi[1:-1] = 0
    return psi * 3


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("kind", ["dense", "sparse", "one", "ends"])
@pytest.mark.parametrize("n,shots", [(1, 5), (7, 300), (12, 4096), (12, 4097), (13, 1), (15, 900),
                                     (22, 400), (23, 5000)])
def test_samples_match_oracle(n, shots, kind, dtype):
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(n * 7 + shots)
    s = qsv.Simulator(n_max=n, dtype=dtype, use_torch_stream=False)
    s.allocate(n)
    psi = state(kind, n, rng).astype(s.np_dtype)
    s.set_state(psi)
    psi = psi.astype(np.complex128)
    u = rng.random(shots)
    u[0] = 0.0
    u[-1] = 1 - 2.0 ** -53
    got, want = s.sample(u), oracle.sample(psi, u)
    p = np.abs(psi) ** 2
    assert np.all(p[got.astype(np.int64)] > 0)
    cdf = np.cumsum(p)
    for k in np.nonzero(got != want)[0]:
        i = int(min(got[k], want[k]))
        assert abs(u[k] * cdf[-1] - cdf[i]) <= 1e-10 * cdf[-1]
    assert np.count_nonzero(got != want) <= 2
    s.close()


def test_samples_of_a_zero_state():
    from paper_1612_08091_amd import qsv
    for n in (3, 14):
        s = qsv.Simulator(n_max=n, use_torch_stream=False)
        s.allocate(n)
        s.set_state(np.zeros(1 << n))
        assert s.sample([0.0, 0.7]).tolist() == [0, 0]
        s.close()
