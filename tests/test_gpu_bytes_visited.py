"""Bytes and operations booked for tile passes: those of the tiles visited.  The
first flush of a state visits the tiles that its gates reach, every later one all of
them, also after a reset."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,elem", [("c128", 16), ("c64", 8)])
def test_first_flush_books_the_tiles_it_visits(dtype, elem):
    from paper_1612_08091_amd import qsv
    n, tile = 18, 1 << 12
    s = qsv.Simulator(n_max=n, dtype=dtype, timing=True, use_torch_stream=False)
    s.allocate(n)

    def booked(qubits):
        before, t = s.stats(), s.kernel_times()["tile"][2]
        for q in qubits:
            s.apply(W.H, [q])
        s.flush()
        after = s.stats()
        assert after["passes"] - before["passes"] == 1
        got = after["alg_bytes"] - before["alg_bytes"]
        assert s.kernel_times()["tile"][2] - t == got
        return got / (2.0 * elem), after["alg_flops"] - before["alg_flops"]

    amps, flops = booked([0, 5])
    assert amps == tile
    full, full_flops = booked([0, 5])
    assert full == 1 << n
    assert full_flops == flops * (1 << n) / tile
    s.reset()
    assert booked([0])[0] == 1 << n
    s.close()
