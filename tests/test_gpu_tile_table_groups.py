"""Runs of diagonal tables that the register-tile kernel reads in one operation,
against the oracle: controlled phases and z rotations on few register bits, with
their other qubits in the lane, the wave, and outside the tile, between gates that
mix (a QFT's pattern), for every tile shape.  On the host model of the kernel
(1e-13) and on the device: n gates of unit norm err by at most a few eps each, so
1e-12 (complex128) and 600 gates x 4 x 6e-8 / 2^(n/2) < 2e-5 (complex64, norm of
the difference below 2e-4)."""
import numpy as np
import pytest

import oracle
import workloads as W

SHAPES = [(11, 3), (12, 3), (12, 4), (13, 4), (13, 5)]


def phases_between_mixes(n, rng):
    c = W.Circuit(n)
    for q in rng.permutation(n).tolist():
        c.add(W.H, (q,))
        for ctl in rng.permutation(n).tolist():
            if ctl == q:
                continue
            if rng.integers(0, 8) == 0:
                other = [x for x in range(n) if x not in (q, ctl)]
                c.add(W.phase(float(rng.uniform(0, 6))), (q,), (ctl, int(rng.choice(other))))
            else:
                c.add(W.phase(float(rng.uniform(0, 6))), (q,), (ctl,))
        c.add(W.rz(float(rng.uniform(0, 6))), (int(rng.integers(0, n)),))
    return c


def run(n, tile_bits, reg_bits, dtype="c128"):
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(31 * n + tile_bits + reg_bits)
    circ = phases_between_mixes(n, rng)
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi /= np.linalg.norm(psi)
    s = qsv.Simulator(n_max=n, mode="tiled", k_max=2, tile_bits=tile_bits, reg_bits=reg_bits,
                      dtype=dtype, use_torch_stream=False)
    s.allocate(n)
    return s, circ, psi


@pytest.mark.parametrize("tile_bits,reg_bits", SHAPES)
@pytest.mark.parametrize("n", [13, 16])
def test_groups_on_the_host_model(n, tile_bits, reg_bits):
    s, circ, psi = run(n, tile_bits, reg_bits)
    s.run(circ)
    got, info = s.check_tile_programs(psi)
    s.close()
    assert info["reg_passes"] == info["passes"] >= 1
    # groups take out a quarter of a pass's ops wherever a pass uses them; a
    # state of one or two tiles has too few tables for it
    if n == 16:
        assert info["instructions"] < 0.75 * (info["diag_ops"] + info["real_ops"] + info["remaps"])
    assert float(np.max(np.abs(got - oracle.run(circ, psi)))) <= 1e-13


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 2e-4)])
@pytest.mark.parametrize("tile_bits,reg_bits", SHAPES)
def test_groups_on_the_device(tile_bits, reg_bits, dtype, tol):
    n = 16
    s, circ, psi = run(n, tile_bits, reg_bits, dtype)
    s.set_state(psi)
    s.run(circ)
    got = s.get_state()
    s.close()
    assert np.linalg.norm(got - oracle.run(circ, psi)) <= tol
