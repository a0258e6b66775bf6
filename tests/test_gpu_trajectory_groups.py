"""Trajectory steps whose waiting gates run in the reduction's pass, against the
oracle: no gate, one and two on the targets and beside them, controls, gates on
exactly three qubits with the targets, on four (flushed on their own), a 3-qubit
gate, targets low, high and in falling order, a state of the targets alone and
one of several sweeps of the grid.  Branches equal, probabilities and state
within 1e-12 (complex128) or 1e-5 (complex64)."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

ONE, TWO = W.amplitude_damping(0.3), [np.kron(a, b) for a in W.depolarizing(0.3) for b in W.dephasing(0.4)]


def cases(n):
    top = n - 1
    yield [], [0], ONE
    yield [([0], [])], [0], ONE
    yield [([top], [])], [0], ONE
    if n > 1:
        yield [([0], [top])], [top], ONE
        yield [([0], []), ([top], [0])], [top, 0], TWO
    if n > 3:
        yield [([0], [top]), ([1], [])], [top], ONE
        yield [([1, 0], [top])], [1], ONE
        yield [([2], [1]), ([1], [])], [2, top], TWO
        yield [([top, 0, 1], [])], [top, 1], TWO
        yield [([0], [1]), ([2], []), ([top], [])], [top], ONE       # four qubits


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 4, 9, 13, 20])
def test_steps_with_waiting_gates(n, dtype):
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(50 + n)
    s = qsv.Simulator(n_max=n, dtype=dtype, use_torch_stream=False)
    s.allocate(n)
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi /= np.linalg.norm(psi)
    s.set_state(psi)
    tol = 1e-12 if dtype == "c128" else 1e-5
    for gates, targets, kraus in cases(n):
        for t, c in gates:
            u = W.haar_unitary(1 << len(t), rng)
            s.apply(u, t, c)
            oracle.apply(psi, u, t, c)
        x = rng.random()
        j, p = s.apply_kraus_sampled(kraus, targets, x)
        want_j, want_p = oracle.kraus_sample(psi, kraus, targets, x)
        assert j == want_j
        assert np.max(np.abs(p - want_p)) <= tol
        assert np.linalg.norm(s.get_amplitudes(range(min(1 << n, 64))) - psi[:64]) <= tol
    assert np.linalg.norm(s.get_state() - psi) <= tol * 10
    s.close()
