"""Measurement of several qubits in one call against the oracle's qubit-by-qubit
measurement: outcomes equal, collapsed state within 1e-12 (complex128, max abs)
or 1e-5 (complex64, norm).  The lists cover the edges of the split: branches
that one workgroup resolves (up to 2^13 amplitudes), one histogram and the rest,
several histograms, qubits below and above the lane bits, decided qubits below
lane bits, a single qubit, and more amplitudes than one sweep of the grid."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

LISTS = {
    "one low": (16, [0]), "one high": (16, [15]), "smallest": (1, [0]),
    "tail only": (13, [3, 12, 0]), "tail edge": (13, list(range(13))),
    "hist edge": (14, list(range(13, -1, -1))),
    "low lanes": (15, [0, 1, 2, 3, 4, 5, 6, 7]), "lane edge": (15, [5, 6, 4, 7]),
    "below lanes": (19, [2, 0, 14, 1, 5, 3, 6, 18, 4]), "high only": (19, [18, 17, 16, 15]),
    "no tail": (20, [19, 0, 7, 3, 11]), "several hists": (22, list(range(21, -1, -1))),
}


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("name", sorted(LISTS))
def test_measure_list_matches_oracle(name, dtype):
    from paper_1612_08091_amd import qsv
    n, qs = LISTS[name]
    rng = np.random.default_rng(n * 100 + len(qs))
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi = psi / np.linalg.norm(psi) * 1.7           # the weights need not sum to 1
    s = qsv.Simulator(n_max=n, dtype=dtype, use_torch_stream=False)
    s.allocate(n)
    s.set_state(psi)
    want = psi.astype(s.np_dtype).astype(np.complex128)
    u = rng.random(len(qs))
    got_bits = s.measure(qs, u)
    assert got_bits == [oracle.measure(want, q, x)[0] for q, x in zip(qs, u)]
    got = s.get_state()
    if dtype == "c128":
        assert np.max(np.abs(got - want)) <= 1e-12
    else:
        assert np.linalg.norm(got - want) <= 1e-5
    assert s.measure(qs, 1 - u) == got_bits          # a branch stays what it is
    s.close()


def test_measure_of_weights_near_the_end_of_the_range():
    """Weights below the range of the joint histogram go qubit by qubit."""
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(5)
    psi = (rng.standard_normal(1 << 6) + 1j * rng.standard_normal(1 << 6)) * 1e-145
    s = qsv.Simulator(n_max=6, use_torch_stream=False)
    s.allocate(6)
    s.set_state(psi)
    u = rng.random(6)
    want = [oracle.measure(psi, q, x)[0] for q, x in enumerate(u)]
    assert s.measure(range(6), u) == want
    assert np.max(np.abs(s.get_state() - psi)) <= 1e-12
    s.set_state(np.zeros(1 << 6))
    with pytest.raises(qsv.QsvError) as ei:
        s.measure([0], [0.5])
    assert ei.value.code == 3
    s.close()
