"""Gates that Simulator.run and DensityMatrix.run hand over in one call, against
the same gates one by one: the plans and their programs are the same, and what
cannot go in a list (a matrix larger than its gate, another dtype or layout, a
qubit that is refused) does what it did in a call of its own, the gates before it
queued."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_1612_08091_amd import qsv



def handle(n):
    s = qsv.Simulator(n_max=n, mode="tiled", use_torch_stream=False)
    s.allocate(n)
    return s


@pytest.mark.parametrize("n,layers", [(12, 1), (13, 4), (16, 12)])
def test_runs_queue_the_same_gates(n, layers):
    rng = np.random.default_rng(n)
    c = W.config1_random(n, layers=layers)
    u = W.haar_unitary(4, rng)
    c.add(u.T, (n - 1, 0))                              # not in C order
    c.add(u.real.astype(np.float32), (0, 1))            # another dtype
    order = rng.permutation(n).tolist()
    a, b = handle(n), handle(n)
    a.run(c, order)
    for g in c.gates:
        b.apply(g.matrix, [order[q] for q in g.targets], [order[q] for q in g.controls])
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    got, want = a.check_tile_programs(psi), b.check_tile_programs(psi)
    assert got[1] == want[1]
    assert np.array_equal(got[0], want[0])
    a.close()
    b.close()


def test_refused_gates_leave_those_before_them():
    rng = np.random.default_rng(4)
    n = 12
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    for bad in ([(W.X, (n,), ())], [(W.X, (1,), (1,))], [(np.full((2, 2), np.inf), (0,), ())],
                [(W.X, (2 ** 40,), ())], [(W.X, (), ())]):
        c = W.Circuit(2)
        for u, t, ctl in [(W.H, (0,), ()), (W.X, (1,), (0,))] + bad + [(W.H, (1,), ())]:
            c.add(u, t, ctl)
        s = handle(n)
        ids = list(range(n)) + [n]
        with pytest.raises((qsv.QsvError, OverflowError, IndexError)):
            s.run(c, ids)
        got, _ = s.check_tile_programs(psi)
        s.close()
        want = psi.copy()
        oracle.apply(want, W.H, (0,), ())
        oracle.apply(want, W.X, (1,), (0,))
        assert np.max(np.abs(got - want)) <= 1e-13


def test_channels_in_a_list():
    rng = np.random.default_rng(6)
    n = 6
    kraus = W.amplitude_damping(0.3)
    ev = [("gate", W.haar_2x2(rng), (0,), ()), ("kraus", kraus, (3,)),
          ("gate", W.X, [1], [4]), ("kraus", tuple(kraus), (5,)),
          ("kraus", np.stack(kraus), [0])]
    a, b = (qsv.DensityMatrix(n, use_torch_stream=False) for _ in range(2))
    a.run(ev)
    for e in ev:
        if e[0] == "gate":
            b.apply(e[1], e[2], e[3])
        else:
            b.channel(e[1], e[2])
    psi = rng.standard_normal(1 << 2 * n) + 1j * rng.standard_normal(1 << 2 * n)
    got, want = a.sim.check_tile_programs(psi), b.sim.check_tile_programs(psi)
    assert got[1] == want[1] and np.array_equal(got[0], want[0])
    for bad in ([], [np.eye(2), np.eye(4)], [np.eye(2) * np.nan]):
        with pytest.raises((qsv.QsvError, ValueError)):
            a.run([("kraus", bad, (0,))])
    a.close()
    b.close()
