"""Results that the host waits for by their values: calls that end while it looks
(small states) and calls whose queue outlasts the look (26 qubits), in turn on two
handles.  The states are uniform superpositions, with known answers: probability
1/2, <X> = 1, sample floor(u 2^n), channel probabilities of a |+> state; 1e-12."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 14, 26])
def test_results(n):
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(n)
    gamma = 0.3
    kraus = W.amplitude_damping(gamma)
    ham = W.PauliSum([1, 1 << (n - 1), 0], [0, 0, 1], [1.0, 0.5, 2.0])
    sims = [qsv.Simulator(n_max=n, use_torch_stream=False) for _ in range(2)]
    for s in sims:
        s.allocate(n)
    for turn in range(3):
        for s in sims:
            s.reset()
            for _ in range(5 if n < 20 else 41):        # an odd number of layers of H
                for q in range(n):
                    s.apply(W.H, (q,))
        for s in sims:
            u = rng.random(50)
            assert abs(s.get_probability([n - 1], [1]) - 0.5) <= 1e-12
            assert abs(s.expectation(ham) - 1.5) <= 1e-11
            got = s.sample(u)
            near = np.abs(u * 2.0 ** n - np.round(u * 2.0 ** n)) < 1e-3
            assert np.array_equal(got[~near], np.floor(u * 2.0 ** n).astype(np.uint64)[~near])
            j, p = s.apply_kraus_sampled(kraus, [0], 0.999)
            assert np.max(np.abs(p - np.array([1 - gamma / 2, gamma / 2]))) <= 1e-12 and j == 1
            assert abs(s.get_probability([0], [0]) - 1.0) <= 1e-12
    for s in sims:
        s.close()
