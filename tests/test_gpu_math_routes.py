"""Math gates on a handle's own state under two and more controls: small states in
one pass over all of them, from 64 MiB only the controlled amplitudes in place (both
sides of the line, by the bytes booked for the kernels; a control on a line's bits
keeps the one pass).  Amplitudes only move: equal to numpy's indexing bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype,ctl,in_place", [
    (9, "c128", [4, 8], False), (21, "c128", [5, 20], False), (22, "c64", [7, 8, 21], False),
    (22, "c128", [9, 21], True), (22, "c128", [3, 4, 12], True), (23, "c64", [4, 22], True),
    (22, "c128", [2, 20], False),
])
def test_own_state(n, dtype, ctl, in_place):
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(n + len(ctl))
    reg = [q for q in range(n) if q not in ctl][1:8]
    kind = np.complex128 if dtype == "c128" else np.complex64
    psi = (rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)).astype(kind)
    tab = rng.permutation(1 << len(reg)).astype(np.uint32)
    s = qsv.Simulator(n_max=n, dtype=dtype, timing=True, use_torch_stream=False)
    s.allocate(n)
    s.set_state(psi)
    s.apply_math(reg, tab, ctl)
    got = s.get_state()
    moved = s.kernel_times()["mono"][2]
    s.close()
    i = np.arange(1 << n, dtype=np.int64)
    x = np.zeros_like(i)
    for b, q in enumerate(reg):
        x |= ((i >> q) & 1) << b
    y = tab[x].astype(np.int64)
    to = i.copy()
    for b, q in enumerate(reg):
        to = (to & ~(1 << q)) | (((y >> b) & 1) << q)
    on = np.all([(i >> q) & 1 for q in ctl], axis=0)
    want = np.empty_like(psi)
    want[np.where(on, to, i)] = psi
    assert np.array_equal(got, want)
    assert moved == psi.nbytes * (4.0 / (1 << len(ctl)) if in_place else 2.0)
