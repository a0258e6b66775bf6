"""The imaginary part of a Pauli sum: 0 for a finite state, whatever the letters;
of a state with an amplitude that is not finite still 0 for strings of Z letters,
and NaN as soon as a string with X letters (0 times infinity in its pairs) or a
coefficient that is not finite takes part."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("n", [2, 9, 14])
def test_imaginary_part(n, value):
    from paper_1612_08091_amd import qsv
    full = (1 << n) - 1
    rng = np.random.default_rng(n)
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi /= np.linalg.norm(psi)
    s = qsv.Simulator(n_max=n, use_torch_stream=False)
    s.allocate(n)
    strings = [(0, full), (1 << (n - 1), 0), (1, 1), (full, 2)]

    def parts(which, coeff):
        x, z = zip(*which)
        return s.get_expectation_complex(x, z, coeff)

    s.set_state(psi)
    for t in strings:
        assert parts([t], [0.7])[1] == 0.0
    assert parts(strings, [1.0, -2.0, 3.0, 0.5])[1] == 0.0
    assert np.isnan(parts(strings[:1], [np.inf])[1])
    psi[1] = value
    s.set_state(psi)
    re, im = parts(strings[:1], [0.7])
    assert not np.isfinite(re) and im == 0.0
    assert parts([(0, 0), (0, 1)], [0.7, 0.1])[1] == 0.0
    for t in strings[1:]:
        re, im = parts([strings[0], t], [0.7, 0.1])
        assert not np.isfinite(re) and np.isnan(im)
    s.close()
