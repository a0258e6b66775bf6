"""Pauli sums against the oracle where the tile plan can go wrong: states
smaller than a tile (padded bits), of one tile and of several; X masks that fill
a tile, fit in none, lie only on the lowest or highest positions or share a
mask with both parities of Y letters; Z strings alone; one term and many (rows
shared out, several tile shapes).  Bound: the value of a string is a sum of
2^n products of size <= 1 in norm, accumulated in double: 1e-12 per unit of
sum |c| (complex128), 1e-5 for a complex64 state rounded from the oracle's."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def masks(kind, n, terms, rng):
    full = (1 << n) - 1
    z = rng.integers(0, full + 1, terms)
    if kind == "z only":
        x = np.zeros(terms, dtype=np.int64)
    elif kind == "low":
        x = rng.integers(0, min(8, full + 1), terms)
    elif kind == "high":
        x = rng.integers(0, min(8, full + 1), terms) << max(n - 3, 0) & full
    elif kind == "shared":
        x = np.full(terms, (1 << (n - 1)) | 1)
    elif kind == "weight":          # from one X letter to more than a tile holds
        x = np.array([sum(1 << int(q) for q in rng.choice(n, 1 + t % n, replace=False))
                      for t in range(terms)])
    else:
        x = rng.integers(0, full + 1, terms)
    return W.PauliSum(x.astype(np.uint64), z.astype(np.uint64), rng.standard_normal(terms))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("kind", ["z only", "low", "high", "shared", "weight", "dense"])
@pytest.mark.parametrize("n,terms", [(1, 3), (4, 40), (9, 30), (11, 7), (12, 25), (13, 1), (16, 60), (18, 12)])
def test_pauli_sums_match_oracle(n, terms, kind, dtype):
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(1000 * n + terms)
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi /= np.linalg.norm(psi)
    ham = masks(kind, n, terms, rng)
    s = qsv.Simulator(n_max=n, dtype=dtype, use_torch_stream=False)
    s.allocate(n)
    s.set_state(psi)
    want, _ = oracle.expectation(psi, ham)
    tol = (1e-12 if dtype == "c128" else 1e-5) * max(1.0, float(np.sum(np.abs(ham.coeff))))
    re, im = s.get_expectation_complex(ham.xmask, ham.zmask, ham.coeff)
    assert abs(re - want) <= tol
    assert im == 0.0
    assert s.get_expectation(ham.xmask, ham.zmask, ham.coeff) == re      # the same on every run
    s.close()


def test_pauli_sum_coefficients_that_are_not_finite():
    from paper_1612_08091_amd import qsv
    s = qsv.Simulator(n_max=3, use_torch_stream=False)
    s.allocate(3)
    s.apply(W.ry(0.4), [0])
    assert s.get_expectation([0, 1], [1, 0], [np.inf, 2.0]) == np.inf
    assert s.get_expectation([0, 1], [1, 0], [1.0, -np.inf]) == -np.inf
    assert np.isnan(s.get_expectation([0, 1], [1, 0], [np.nan, 2.0]))
    assert s.get_expectation([], [], []) == 0.0
    s.close()
