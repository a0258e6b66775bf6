"""A channel step that applies the waiting gates on the way returns with the state
written: the borrowed buffer, read at once on a stream that has not waited for the
handle's, holds U psi.  (The channel is the identity, whose branch stays queued.)
Groups of one to three qubits, states of one workgroup to thousands; an amplitude
is a sum of at most 8 products below 1: 1e-14 and 1e-6 are several times its
rounding."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def apply(psi, u, qubits):
    """u (bit j of its index = qubits[j]) on a state, in 64 bits."""
    n, k = psi.numel().bit_length() - 1, len(qubits)
    axes = [n - 1 - q for q in reversed(qubits)]
    rest = [a for a in range(n) if a not in axes]
    t = psi.reshape((2,) * n).permute(axes + rest).reshape(1 << k, -1)
    t = torch.as_tensor(u, dtype=torch.complex128, device=psi.device) @ t
    back = np.argsort(axes + rest).tolist()
    return t.reshape((2,) * n).permute(back).reshape(-1)


@pytest.mark.parametrize("dtype,tol", [("c128", 1e-14), ("c64", 1e-6)])
@pytest.mark.parametrize("n", [8, 17, 24])
def test_state_is_written_when_the_call_returns(n, dtype, tol):
    from paper_1612_08091_amd import qsv
    rng = np.random.default_rng(n)
    kind = torch.complex128 if dtype == "c128" else torch.complex64
    buf = torch.empty(1 << n, dtype=kind, device="cuda")
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    sim = qsv.Simulator(n_max=n, dtype=dtype, state=buf, stream=own.cuda_stream)
    sim.allocate(n)
    g = torch.Generator(device="cuda").manual_seed(n)
    for qubits in ([2], [n - 1, 0], [1, n - 2, 4]):
        psi = torch.view_as_complex(torch.randn(1 << n, 2, dtype=torch.float64, device="cuda", generator=g))
        psi /= torch.linalg.vector_norm(psi)
        psi = psi.to(kind).to(torch.complex128)
        u = W.haar_unitary(1 << len(qubits), rng)
        want = apply(psi, u, qubits)
        sim.reset()
        sim.state_pointer()
        torch.cuda.synchronize()        # the reset has filled the buffer
        buf.copy_(psi)
        torch.cuda.synchronize()
        sim.apply(u, qubits)
        sim.apply_kraus_sampled([np.eye(2)], qubits[:1], 0.5)
        with torch.cuda.stream(other):
            got = buf.clone()
        other.synchronize()
        assert float((got - want).abs().max()) <= tol, qubits
    sim.close()
