"""The work that a user of the simulator has it do, as cases to time.

Each case is one call sequence through the public entry points of
paper_1612_08091_amd, on inputs made from a seed: circuits run on a state and
read out (samples, Pauli sums, measurement), Pauli sums of a state at hand,
noise as density matrices and as trajectories, emulated arithmetic, adjoint
gradients and batches of small circuits.  ``exact`` gives the same results in
64 bits from plain torch, one gate at a time, without the package.

Qubit j is bit j of the amplitude index; gates act on |0...0> unless said.
"""
import math

import numpy as np
import torch

from paper_1612_08091_amd import qsv

C128, C64 = "c128", "c64"
TORCH_DTYPE = {C128: torch.complex128, C64: torch.complex64}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # The paper's first example: entangle a few qubits, read samples.  The
        # smallest call there is: launches, uploads and waits are all of it.
        {"name": "entangle_5q", "kind": "circuit", "circuit": "ghz", "n": 5, "layers": 1,
         "dtype": C128, "terms": 0, "shots": 100},
        # A random circuit of the size that fits a cache: 16 qubits, 20 layers,
        # 470 gates, 1000 samples, as a development loop runs it.
        {"name": "brick_16q", "kind": "circuit", "circuit": "cnot", "n": 16, "layers": 20,
         "dtype": C128, "terms": 0, "shots": 1000},
        # The headline workload at its full size (16 GiB of state), with the
        # benchmark's read-outs; 10 of its 40 layers, which repeat.
        {"name": "brick_30q", "kind": "circuit", "circuit": "cnot", "n": 30, "layers": 10,
         "dtype": C128, "terms": 8, "shots": 1000},
        # Single precision, as users take it for twice the qubits' room: CZ
        # brick on 28 qubits (2 GiB).
        {"name": "brick_28q_c64", "kind": "circuit", "circuit": "cz", "n": 28, "layers": 20,
         "dtype": C64, "terms": 0, "shots": 0},
        # QFT of a basis state: runs of controlled phases on an odd size.
        {"name": "qft_27q", "kind": "circuit", "circuit": "qft", "n": 27, "layers": 1,
         "dtype": C128, "terms": 0, "shots": 0},
        # A few gates, then the whole register is measured, as at the end of
        # the paper's algorithms; returns the collapsed state.
        {"name": "measure_25q", "kind": "measure", "n": 25, "m": 25, "layers": 2, "dtype": C128},
        # Energy of a state at hand: 200 Pauli strings of weight 1 to 4 (the
        # size of a chemistry or lattice Hamiltonian).
        {"name": "pauli_25q", "kind": "pauli", "n": 25, "terms": 200, "weight": 4, "dtype": C128},
        # <H> and its gradient over the angles of a hardware-efficient ansatz:
        # one optimiser step of a variational program.
        {"name": "adjoint_20q", "kind": "adjoint", "n": 20, "layers": 8, "terms": 100,
         "weight": 4, "dtype": C128},
        # Many small circuits with their own dense Pauli sums at once, the
        # batched form (states of 8 to 20 qubits, single precision).
        {"name": "batch_192", "kind": "batch", "count": 192, "n_lo": 8, "n_hi": 20, "layers": 6,
         "terms": 64, "dtype": C64},
        # A noisy circuit as a density matrix: 12 qubits, a 24-qubit vector.
        {"name": "density_12q", "kind": "density", "n": 12, "layers": 4, "dtype": C128},
        # The same noise as one stochastic trajectory: a reduction, a host
        # decision and a gate per channel, on a 16-qubit state.
        {"name": "trajectory_16q", "kind": "trajectory", "n": 16, "layers": 4, "dtype": C128},
        # Emulated arithmetic: a layer of gates, then the controlled modular
        # multiplication of Shor's algorithm on 20 of 27 qubits.
        {"name": "modmul_27q", "kind": "math", "n": 27, "w": 20, "controls": 1, "mul": True,
         "dtype": C128},
    ]


def draw(rng):
    kind = rng.choice(["circuit"] * 5 + ["measure", "pauli", "adjoint", "batch", "density",
                                         "trajectory", "math"])
    dtype = rng.choice([C128, C128, C64])
    if kind == "circuit":
        circ = rng.choice(["ghz", "cnot", "cnot", "cz", "hea", "qft"])
        n = rng.randint(3, 28)
        # samples and sums of a rounded state are whole numbers and 64-bit
        # values: they are asked of double-precision states
        shots = rng.choice([0, 1, 37, 1000]) if dtype == C128 and n <= 26 else 0
        return {"kind": kind, "circuit": circ, "n": n, "dtype": dtype, "shots": shots,
                "layers": rng.randint(1, 20),
                # (sums that are zero by symmetry, as those of a QFT state, say nothing)
                "terms": rng.choice([0, 1, 8, 30]) if dtype == C128 and circ in ("cnot", "cz", "hea") else 0}
    if kind == "measure":
        n = rng.randint(4, 26)
        return {"kind": kind, "n": n, "m": rng.choice([1, n // 2, n]), "layers": rng.randint(1, 4),
                "dtype": dtype}
    if kind == "pauli":
        n = rng.randint(6, 26)
        return {"kind": kind, "n": n, "terms": int(2 ** rng.uniform(0, 7.9)),
                "weight": rng.choice([1, 2, 4, 4, min(n, 12)]), "dtype": dtype}
    if kind == "adjoint":
        return {"kind": kind, "n": rng.randint(4, 22), "layers": rng.randint(1, 8),
                "terms": int(2 ** rng.uniform(0, 7)), "weight": rng.choice([1, 2, 4]),
                "dtype": C128}
    if kind == "batch":
        lo = rng.randint(3, 12)
        return {"kind": kind, "count": int(2 ** rng.uniform(4, 7.5)), "n_lo": lo,
                "n_hi": rng.randint(lo, 20), "layers": rng.randint(1, 6),
                "terms": int(2 ** rng.uniform(2, 6)), "dtype": rng.choice([C64, C64, C128])}
    if kind == "density":
        return {"kind": kind, "n": rng.randint(2, 13), "layers": rng.randint(1, 4), "dtype": dtype}
    if kind == "trajectory":
        return {"kind": kind, "n": rng.randint(3, 20), "layers": rng.randint(1, 4), "dtype": C128}
    n = rng.randint(6, 27)
    c = rng.randint(0, 2)
    return {"kind": kind, "n": n, "w": rng.randint(2, min(22, n - c)), "controls": c,
            "mul": rng.choice([True, False]), "dtype": dtype}


# ------------------------------------------------------------------ generators
class Gate:
    def __init__(self, matrix, targets, controls=(), param=-1, axis=""):
        self.matrix = np.asarray(matrix, dtype=np.complex128)
        self.targets, self.controls = tuple(targets), tuple(controls)
        self.param, self.axis = param, axis


class Circuit:
    def __init__(self, n, theta=None):
        self.n, self.gates, self.theta = n, [], theta

    def add(self, *a, **k):
        self.gates.append(Gate(*a, **k))


class PauliSum:
    def __init__(self, x, z, c):
        self.xmask, self.zmask = np.array(x, dtype=np.uint64), np.array(z, dtype=np.uint64)
        self.coeff = np.array(c, dtype=np.float64)


_H = np.array([[1, 1], [1, -1]]) / math.sqrt(2)
_X, _Y, _Z = np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]]), np.diag([1.0, -1.0])
_SWAP = np.eye(4)[[0, 2, 1, 3]]


def _haar(rng):
    q, r = np.linalg.qr(rng.standard_normal((2, 2)) + 1j * rng.standard_normal((2, 2)))
    d = np.diagonal(r)
    return q * (d / np.abs(d))[None, :]


def _ry(t):
    return np.array([[math.cos(t / 2), -math.sin(t / 2)], [math.sin(t / 2), math.cos(t / 2)]])


def _rz(t):
    return np.diag([np.exp(-0.5j * t), np.exp(0.5j * t)])


def _pairs(n, layer):
    return [(q, q + 1) for q in range(layer % 2, n - 1, 2)]


def _hea(n, layers, rng):
    th = rng.uniform(0, 2 * math.pi, 2 * n * layers)
    c = Circuit(n, th)
    for layer in range(layers):
        for q in range(n):
            p = 2 * (layer * n + q)
            c.add(_ry(th[p]), (q,), (), p, "Y")
            c.add(_rz(th[p + 1]), (q,), (), p + 1, "Z")
        for q in range(n - 1):
            c.add(_Z, (q + 1,), (q,))
    return c


def _circuit(kind, n, layers, rng):
    if kind == "hea":
        return _hea(n, layers, rng)
    c = Circuit(n)
    if kind == "ghz":           # a rotation instead of H: its weights are the seed's
        c.add(_ry(rng.uniform(0.5, 2.5)), (0,))
        for q in range(1, n):
            c.add(_X, (q,), (0,))
    elif kind == "qft":         # of the basis state |x>
        c.x = int(rng.integers(1, 1 << n))
        for q in range(n):
            if (c.x >> q) & 1:
                c.add(_X, (q,))
        for j in range(n - 1, -1, -1):
            c.add(_H, (j,))
            for k in range(j - 1, -1, -1):
                c.add(np.diag([1, np.exp(1j * math.pi / 2 ** (j - k))]), (j,), (k,))
        for i in range(n // 2):
            c.add(_SWAP, (i, n - 1 - i))
    else:                       # brick: Haar on every qubit, CNOT or CZ on pairs
        for layer in range(layers):
            for q in range(n):
                c.add(_haar(rng), (q,))
            for a, b in _pairs(n, layer):
                c.add(_X if kind == "cnot" else _Z, (b,), (a,))
    return c


def _local_paulis(n, terms, weight, rng):
    xs, zs = [], []
    for _ in range(terms):
        w = int(rng.integers(1, min(weight, n) + 1))
        x = z = 0
        for q, p in zip(rng.choice(n, w, replace=False), rng.integers(0, 3, w)):
            x |= int(p != 2) << int(q)
            z |= int(p != 0) << int(q)
        xs.append(x)
        zs.append(z)
    return PauliSum(xs, zs, rng.standard_normal(terms))


def _dense_paulis(n, terms, rng):
    m = rng.integers(0, 1 << n, (2, terms))
    return PauliSum(m[0], m[1], rng.standard_normal(terms))


def _noisy(n, layers, rng):
    """("gate", U, targets, controls) and ("kraus", [K], targets) of a noisy brick."""
    p = g = 1e-2
    dep = [math.sqrt(1 - 3 * p / 4) * np.eye(2)] + [math.sqrt(p / 4) * m for m in (_X, _Y, _Z)]
    damp = [np.diag([1, math.sqrt(1 - g)]), np.array([[0, math.sqrt(g)], [0, 0]])]
    ev = []
    for layer in range(layers):
        for q in range(n):
            ev.append(("gate", _haar(rng), (q,), ()))
            ev.append(("kraus", dep, (q,)))
        for a, b in _pairs(n, layer):
            ev.append(("gate", _X, (b,), (a,)))
            ev += [("kraus", dep, (a,)), ("kraus", dep, (b,)), ("kraus", damp, (b,))]
    return ev


def _inputs(case, seed):
    """Everything of a case that the seed decides, apart from random states."""
    rng = np.random.Generator(np.random.PCG64([int(seed), 161208091]))
    k, s = case["kind"], {}
    if k in ("circuit", "measure"):
        s["circ"] = _circuit(case.get("circuit", "cnot"), case["n"], case["layers"], rng)
        if k == "measure":
            s["qubits"] = [int(q) for q in rng.permutation(case["n"])[: case["m"]]]
            s["u"] = rng.random(case["m"])
        else:
            s["ham"] = _local_paulis(case["n"], case["terms"], 4, rng) if case["terms"] else None
            s["u"] = rng.random(case["shots"])
    elif k == "pauli":
        s["ham"] = _local_paulis(case["n"], case["terms"], case["weight"], rng)
    elif k == "adjoint":
        s["circ"] = _hea(case["n"], case["layers"], rng)
        s["ham"] = _local_paulis(case["n"], case["terms"], case["weight"], rng)
    elif k == "batch":
        ns = rng.integers(case["n_lo"], case["n_hi"] + 1, case["count"])
        s["circs"] = [_hea(int(n), case["layers"], rng) for n in ns]
        s["hams"] = [_dense_paulis(int(n), case["terms"], rng) for n in ns]
    elif k == "density":
        s["events"] = _noisy(case["n"], case["layers"], rng)
        s["ham"] = _local_paulis(case["n"], 10, 2, rng)
    elif k == "trajectory":
        s["events"] = _noisy(case["n"], case["layers"], rng)
        s["u"] = rng.random(sum(e[0] == "kraus" for e in s["events"]))
    else:                       # controls, then the register, on neighbouring qubits
        n, w, c = case["n"], case["w"], case["controls"]
        s["circ"] = _circuit("cnot", n, 1, rng)
        at = int(rng.integers(0, n - w - c + 1))
        s["reg"], s["ctl"] = list(range(at + c, at + c + w)), list(range(at, at + c))
        size = np.uint64(1 << w)
        x = np.arange(1 << w, dtype=np.uint64)
        if case["mul"]:         # x -> a x mod N below an odd N, a prime to it
            mod = int(size) - 1
            a = int(rng.integers(1, mod + 1))
            while math.gcd(a, mod) != 1:
                a = a % mod + 1
            s["table"] = np.where(x < mod, x * np.uint64(a) % np.uint64(mod), x).astype(np.uint32)
        else:
            s["table"] = ((x + np.uint64(rng.integers(1, 1 << w))) % size).astype(np.uint32)
    return s


def _random_state(n, dtype, seed, dev="cuda"):
    """A random normalised state, as deep circuits leave it."""
    g = torch.Generator(device=dev).manual_seed(int(seed) & 0x7FFFFFFF)
    v = torch.randn(1 << n, 2, dtype=torch.float64, device=dev, generator=g)
    v /= torch.linalg.vector_norm(v)
    return torch.view_as_complex(v).to(TORCH_DTYPE[dtype])


# ------------------------------------------------------------------ the passes
def _simulator(n, dtype):
    """A simulator on a torch buffer, so that the program holds its state."""
    buf = torch.empty(1 << n, dtype=TORCH_DTYPE[dtype], device="cuda")
    sim = qsv.Simulator(n_max=n, dtype=dtype, state=buf)
    sim.allocate(n)
    return sim, buf


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"], k = case, case["kind"]
    if k == "batch":
        s["batch"] = qsv.Batch(s["circs"], s["hams"], dtype=case["dtype"], autotune=False)
    elif k == "density":
        n = case["n"]
        s["buf"] = torch.empty(1 << 2 * n, dtype=TORCH_DTYPE[case["dtype"]], device="cuda")
        s["rho"] = qsv.DensityMatrix(n, dtype=case["dtype"], state=s["buf"])
    elif k == "adjoint":
        s["sim"] = qsv.Simulator(n_max=case["n"], dtype=case["dtype"])
    else:
        s["sim"], s["buf"] = _simulator(case["n"], case["dtype"])
        if k == "pauli":                # the state is what the program has in hand
            s["sim"].state_pointer()
            s["buf"].copy_(_random_state(case["n"], case["dtype"], seed))
    return s


def run(s):
    k, case = s["case"]["kind"], s["case"]
    if k == "batch":
        e = s["batch"].run()
        return e if case["dtype"] == C128 else e.astype(np.float32)     # of complex64 states
    if k == "density":
        s["rho"].sim.reset()
        s["rho"].run(s["events"])
        s["rho"].flush()
        p = s["rho"].probabilities()
        if case["dtype"] == C64:                # a complex64 state's probabilities
            return {"rho": s["buf"], "p": p.astype(np.float32)}
        return {"rho": s["buf"], "p": p, "e": s["rho"].expectation(s["ham"])}
    sim = s["sim"]
    if k == "adjoint":
        e, g = qsv.adjoint_gradient(sim, s["circ"], s["ham"])
        return {"e": e, "grad": g}
    if k == "pauli":
        return sim.expectation(s["ham"])
    sim.reset()
    if k == "trajectory":
        chosen, probs, i = [], [], 0
        for ev in s["events"]:
            if ev[0] == "gate":
                sim.apply(ev[1], ev[2], ev[3])
            else:
                j, p = sim.apply_kraus_sampled(ev[1], ev[2], s["u"][i])
                chosen.append(j)
                probs.append(p)
                i += 1
        sim.flush()
        return {"state": s["buf"], "chosen": np.array(chosen), "p": np.concatenate(probs)}
    sim.run(s["circ"])
    if k == "math":
        sim.apply_math(s["reg"], s["table"], s["ctl"])
        return s["buf"]
    if k == "measure":
        bits = sim.measure(s["qubits"], s["u"])
        return {"state": s["buf"], "bits": np.array(bits)}
    sim.flush()
    out = {"state": s["buf"]}
    if s["ham"] is not None:
        out["norm"] = sim.norm2()
        out["e"] = sim.expectation(s["ham"])
    if len(s["u"]):
        out["samples"] = sim.sample(s["u"]).astype(np.int64)
    return out


def work(case):
    """Each input read once, each output written once; the arithmetic of the
    gates as they are given (14 per amplitude of a dense 1-qubit gate)."""
    k, el = case["kind"], 16 if case["dtype"] == C128 else 8
    if k == "batch":
        dims = [2 ** n for n in range(case["n_lo"], case["n_hi"] + 1)]
        mean_n = (case["n_lo"] + case["n_hi"]) / 2
        amps = case["count"] * sum(dims) / len(dims)
        return {"bytes": case["count"] * (16 * mean_n * case["layers"] + 24 * case["terms"] + 8),
                "flops": amps * (14.0 * mean_n * case["layers"] + 8.0 * case["terms"])}
    n = case["n"]
    dim = 2.0 ** n
    if k == "pauli":
        return {"bytes": dim * el, "flops": 8.0 * dim * case["terms"]}
    if k == "math":
        return {"bytes": dim * el + 4.0 * 2 ** case["w"], "flops": 14.0 * dim * n}
    if k == "adjoint":      # forward, H psi, and the reverse sweep on two vectors
        return {"bytes": 16.0 * 2 * n * case["layers"] + 24 * case["terms"],
                "flops": dim * (3 * 20.0 * n * case["layers"] + 8.0 * case["terms"])}
    if k == "density":      # a gate on rows and columns, a 4 x 4 channel
        d2 = dim * dim
        return {"bytes": d2 * el + 8 * dim,
                "flops": d2 * case["layers"] * (28.0 * n + 30.0 * (n + 1.5 * (n - 1)))}
    if k == "trajectory":
        return {"bytes": dim * el, "flops": dim * case["layers"] * (28.0 * n + 30.0 * n)}
    if k == "measure":
        return {"bytes": dim * el, "flops": dim * (14.0 * n * case["layers"] + 4.0)}
    c = case["circuit"]
    gates = {"ghz": 1, "qft": n * (14 + 1.5 * (n - 1) / 2) / 14.0}.get(c, n * case["layers"])
    return {"bytes": dim * el + 16.0 * case["shots"], "flops": 14.0 * dim * gates}


# ---------------------------------------------------------- the same in 64 bits
def _apply(psi, u, targets, controls=()):
    """One gate on the vector psi, in place: slices of its 2^k amplitudes per group."""
    qs = sorted(list(targets) + list(controls), reverse=True)
    dims, last = [], psi.numel().bit_length() - 1
    for q in qs:
        dims += [1 << (last - q - 1), 2]
        last = q
    v = psi.view(dims + [1 << last])
    at = {q: 2 * i + 1 for i, q in enumerate(qs)}

    def part(r):
        ix = [slice(None)] * v.dim()
        for c in controls:
            ix[at[c]] = 1
        for j, t in enumerate(targets):
            ix[at[t]] = (r >> j) & 1
        return v[tuple(ix)]

    d = len(u)
    rows = [r for r in range(d) if any(u[r][c] != (r == c) for c in range(d))]
    new = []
    for r in rows:
        acc = None
        for c in range(d):
            if u[r][c] != 0:
                acc = part(c) * complex(u[r][c]) if acc is None else acc.add_(part(c), alpha=complex(u[r][c]))
        new.append(acc)
    for r, y in zip(rows, new):
        part(r).copy_(y) if y is not None else part(r).zero_()


def _signs(n, z, dev):
    """(-1)^popcount(j & z) for j < 2^n."""
    s = torch.ones(1, dtype=torch.float64, device=dev)
    for q in range(n):
        s = torch.cat([s, -s if (z >> q) & 1 else s])
    return s


def _pauli(psi, x, z):
    """P psi: psi_j goes to j ^ x with i^(number of Y) (-1)^popcount(j & z)."""
    n = psi.numel().bit_length() - 1
    out = psi * _signs(n, z, psi.device)
    for q in range(n):
        if (x >> q) & 1:
            out = out.view(-1, 2, 1 << q).flip(1).reshape(-1)
    return out.mul_(1j ** (bin(x & z).count("1") % 4))


def _terms(ham):
    return [(int(x), int(z), float(c)) for x, z, c in zip(ham.xmask, ham.zmask, ham.coeff)]


def _energy(psi, ham):
    return sum(c * float(torch.vdot(psi, _pauli(psi, x, z)).real) for x, z, c in _terms(ham))


def _zero_state(n):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[0] = 1
    return psi


def _run_exact(circ):
    psi = _zero_state(circ.n)
    for g in circ.gates:
        _apply(psi, g.matrix, g.targets, g.controls)
    return psi


def _exact_qft(n, x):
    y = torch.arange(1 << n, dtype=torch.int64, device="cuda")
    ang = ((y * x) & ((1 << n) - 1)).double() * (2 * math.pi / (1 << n))
    return torch.polar(torch.full_like(ang, 2.0 ** (-n / 2)), ang)


def _exact_gradient(circ, ham):
    psi = _run_exact(circ)
    phi = torch.zeros_like(psi)
    for x, z, c in _terms(ham):
        phi.add_(_pauli(psi, x, z), alpha=c)
    e, grad = float(torch.vdot(psi, phi).real), np.zeros(len(circ.theta))
    for g in reversed(circ.gates):
        if g.param >= 0:
            q = 1 << g.targets[0]
            x, z = {"X": (q, 0), "Y": (q, q), "Z": (0, q)}[g.axis]
            grad[g.param] += float(torch.vdot(phi, _pauli(psi, x, z)).imag)
        for v in (psi, phi):
            _apply(v, g.matrix.conj().T, g.targets, g.controls)
    return {"e": e, "grad": grad}


def _exact_density(case, s):
    n = case["n"]
    rho = _zero_state(2 * n)
    for ev in s["events"]:
        if ev[0] == "gate":
            _apply(rho, ev[1], ev[2], ev[3])
            _apply(rho, ev[1].conj(), [t + n for t in ev[2]], [c + n for c in ev[3]])
        else:
            t = ev[2][0]
            _apply(rho, sum(np.kron(np.conj(k), k) for k in ev[1]), (t, t + n))
    m = rho.view(1 << n, 1 << n)        # [column][row]
    r, e = torch.arange(1 << n, device="cuda"), 0.0
    for x, z, c in _terms(s["ham"]):    # Tr(rho P)
        tr = (m[r ^ x, r] * _signs(n, z, "cuda")).sum()
        e += c * complex(tr * 1j ** (bin(x & z).count("1") % 4)).real
    return {"rho": rho, "p": torch.diagonal(m).real.clone(),
            **({"e": e} if case["dtype"] == C128 else {})}


def _exact_trajectory(case, s):
    psi, probs, i = _zero_state(case["n"]), [], 0
    for ev in s["events"]:
        if ev[0] == "gate":
            _apply(psi, ev[1], ev[2], ev[3])
            continue
        v = psi.view(-1, 2, 1 << ev[2][0])
        a, b = v[:, 0].reshape(-1), v[:, 1].reshape(-1)
        ab = complex(torch.vdot(b, a))
        rho = np.array([[float(torch.vdot(a, a).real), ab], [np.conj(ab), float(torch.vdot(b, b).real)]])
        p = [max(0.0, float(np.trace(k @ rho @ np.conj(k).T).real)) for k in ev[1]]
        j = next((j for j in range(len(p)) if sum(p[: j + 1]) > s["u"][i] * sum(p)), len(p) - 1)
        _apply(psi, ev[1][j] / math.sqrt(p[j]), ev[2])
        probs += p
        i += 1
    return {"state": psi, "chosen": None, "p": np.array(probs)}


def _exact_measure(case, s):
    psi = _run_exact(s["circ"])
    for q, u in zip(s["qubits"], s["u"]):
        v = psi.view(-1, 2, 1 << q)
        p = [float(torch.linalg.vector_norm(v[:, b]) ** 2) for b in (0, 1)]
        b = 0 if u * (p[0] + p[1]) < p[0] else 1
        v[:, 1 - b] = 0
        psi /= math.sqrt(p[b])
    return {"state": psi, "bits": None}


def exact(case, seed):
    s, k = _inputs(case, seed), case["kind"]
    if k == "pauli":
        return _energy(_random_state(case["n"], case["dtype"], seed).to(torch.complex128), s["ham"])
    if k == "math":
        psi = _run_exact(s["circ"])
        j = torch.arange(1 << case["n"], dtype=torch.int64, device="cuda")
        at, w = s["reg"][0], case["w"]
        new = torch.from_numpy(s["table"].astype(np.int64)).cuda()[(j >> at) & ((1 << w) - 1)]
        new = (j & ~(((1 << w) - 1) << at)) | (new << at)
        ctl = sum(1 << c for c in s["ctl"])
        out = torch.empty_like(psi)
        out[torch.where((j & ctl) == ctl, new, j)] = psi
        return out
    if k == "adjoint":
        return _exact_gradient(s["circ"], s["ham"])
    if k == "batch":
        return np.array([_energy(_run_exact(c), h) for c, h in zip(s["circs"], s["hams"])],
                        dtype=np.float64)
    if k == "density":
        return _exact_density(case, s)
    if k == "trajectory":
        return _exact_trajectory(case, s)
    if k == "measure":
        return _exact_measure(case, s)
    psi = _exact_qft(case["n"], s["circ"].x) if case["circuit"] == "qft" else _run_exact(s["circ"])
    out = {"state": psi}
    if s["ham"] is not None:
        out["norm"], out["e"] = float(torch.linalg.vector_norm(psi) ** 2), _energy(psi, s["ham"])
    if len(s["u"]):
        out["samples"] = None
    return out
