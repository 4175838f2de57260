"""What a program that simulates circuits with this library spends its time on, as cases that can be
timed: gate instructions, variational steps (energy and every gradient) on one state, on a batch of
states and on a list of unlike circuits, forward sweeps, energies, time evolution, the QFT and sampling.

A case is a dict of plain values. `prepare` makes what a program holds before the call: the register, the
angles, and the handles (circuit, observable, and for a list of circuits its registers) that it builds
once and calls with new angles again and again, so those are kept per structure over all seeds. `run`
is one call sequence through paper_1912_10877_amd.binding. `exact` is the same result in complex128 with
torch, from the gate lists below alone.

Energies and gradients are double arrays in the library's interface; those of complex64 registers carry
float precision and come back as float32.
"""
import functools
import math

import numpy as np
import torch

from paper_1912_10877_amd import binding as yb

DTYPES = {"c64": (yb.C64, torch.complex64, 8), "c128": (yb.C128, torch.complex128, 16)}


# ---- the cases ------------------------------------------------------------------------------


def listed():
    return [
        # Single instructions on a small register (the paper's gate benchmark: X, H, T, Rx, CNOT,
        # Toffoli, n from 4 to 25): a call's latency.
        dict(name="instr_10q_c128", kind="instr", n=10, batch=1, dtype="c128"),
        # The smallest usual variational step: 10 qubits, depth 5, 150 gradients.
        dict(name="vqe_10q_d5_c128", kind="vqe", n=10, depth=5, batch=1, dtype="c128"),
        # A middle-sized step, the size most studies of variational circuits use.
        dict(name="vqe_15q_d10_c64", kind="vqe", n=15, depth=10, batch=1, dtype="c64"),
        # The headline: 20 qubits, depth 20, 1200 gradients.
        dict(name="vqe_20q_d20_c64", kind="vqe", n=20, depth=20, batch=1, dtype="c64"),
        # The same circuit on a batched register of 64 states.
        dict(name="vqe_20q_d20_b64_c64", kind="vqe", n=20, depth=20, batch=64, dtype="c64"),
        # A list of unlike small and middle circuits (a sweep over sizes and depths), one call.
        dict(name="uneven_96_c64", kind="uneven", ncirc=96, nmin=8, nmax=20, dmin=4, dmax=16, sizes=4, dtype="c64"),
        # A layered circuit applied once to a large register.
        dict(name="forward_25q_d20_c64", kind="forward", circ="hea", n=25, depth=20, batch=1, dtype="c64"),
        # A random circuit (Haar one-qubit layers, CZ on random pairs), double precision.
        dict(name="random_24q_d16_c128", kind="forward", circ="random", n=24, depth=16, batch=1, dtype="c128"),
        # The energy of a large register under the Heisenberg chain.
        dict(name="energy_25q_c64", kind="energy", ham="heisenberg", terms=0, n=25, batch=1, dtype="c64", hpsi=False),
        # Hamiltonian evolution, the size of the paper's listing.
        dict(name="evolve_16q_c128", kind="evolve", ham="heisenberg", terms=0, n=16, batch=1, dtype="c128", t=0.1),
        # The Fourier transform of a large register.
        dict(name="qft_25q_c128", kind="qft", n=25, k=25, batch=1, dtype="c128", inverse=False, focus=False),
        # A million shots of all the qubits of a large register.
        dict(name="measure_24q_1m_c128", kind="measure", n=24, k=24, batch=1, shots=1 << 20, dtype="c128"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["instr", "vqe", "vqe", "vqe", "uneven", "forward", "forward", "energy", "energy", "evolve", "qft",
                       "measure", "shift"])
    dt = rng.choice(["c64", "c128"])
    big = 25 if dt == "c64" else 24
    if kind == "instr":
        n = rng.randint(4, big)
        return dict(kind=kind, n=n, batch=_log_int(rng, 1, max(1, min(64, 1 << (big - n)))), dtype=dt)
    if kind == "vqe":
        n = rng.randint(5, 20)
        batch = _log_int(rng, 1, max(1, min(128, 1 << (24 - n)))) if rng.random() < 0.4 else 1
        return dict(kind=kind, n=n, depth=rng.randint(2, 20), batch=batch, dtype=dt)
    if kind == "uneven":
        nmin = rng.randint(6, 12)
        return dict(kind=kind, ncirc=_log_int(rng, 6, 80), nmin=nmin, nmax=min(19, nmin + rng.randint(2, 9)), dmin=2,
                    dmax=rng.randint(4, 14), sizes=rng.randint(0, 1 << 20), dtype=dt)
    if kind == "forward":
        circ = rng.choice(["hea", "random"])
        return dict(kind=kind, circ=circ, n=rng.randint(8, big), depth=rng.randint(2, 20), batch=1, dtype=dt)
    if kind == "energy":
        n = rng.randint(6, big)
        ham = rng.choice(["heisenberg", "random"])
        return dict(kind=kind, ham=ham, terms=0 if ham == "heisenberg" else _log_int(rng, 4, 120), n=n,
                    batch=_log_int(rng, 1, max(1, min(64, 1 << (big - n)))) if rng.random() < 0.3 else 1, dtype=dt,
                    hpsi=rng.random() < 0.3)
    if kind == "evolve":
        ham = rng.choice(["heisenberg", "random"])
        return dict(kind=kind, ham=ham, terms=0 if ham == "heisenberg" else _log_int(rng, 4, 60), n=rng.randint(6, 20),
                    batch=1, dtype=dt, t=round(rng.uniform(0.02, 0.2), 3))
    if kind == "qft":
        n = rng.randint(6, big)
        k = n if rng.random() < 0.5 else rng.randint(2, n)
        return dict(kind=kind, n=n, k=k, batch=1, dtype=dt, inverse=rng.random() < 0.5, focus=k < n and rng.random() < 0.5)
    if kind == "measure":
        n = rng.randint(6, big - 1)
        return dict(kind=kind, n=n, k=n if rng.random() < 0.5 else rng.randint(1, n), batch=1, shots=_log_int(rng, 1, 1 << 20),
                    dtype=dt)
    return dict(kind="shift", n=rng.randint(4, 12), depth=rng.randint(1, 5), batch=1, dtype=dt)


# ---- circuits, observables, sizes (plain data, from the case alone) ---------------------------

# A gate is (kind, target, controls, parameter index or -1, 2x2 matrix or None).


@functools.lru_cache(maxsize=256)
def _gates(circ, n, depth):
    gates, p = [], 0
    if circ == "hea":  # Rx.Rz.Rx on every qubit, then the CNOT chain
        for _ in range(depth):
            for q in range(n):
                for kind in ("Rx", "Rz", "Rx"):
                    gates.append((kind, q, (), p, None))
                    p += 1
            for i in range(n - 1):
                gates.append(("X", i + 1, (i,), -1, None))
        return gates, p
    rng = np.random.default_rng(1000 * n + depth)
    for _ in range(depth):  # Haar SU(2) on every qubit, then CZ on random pairs
        for q in range(n):
            v = rng.standard_normal(4)
            v /= np.linalg.norm(v)
            a, b = complex(v[0], v[1]), complex(v[2], v[3])
            gates.append(("dense", q, (), -1, np.array([[a, -b.conjugate()], [b, a.conjugate()]])))
        order = rng.permutation(n)
        for m in range(n // 2):
            gates.append(("Z", int(order[2 * m + 1]), (int(order[2 * m]),), -1, None))
    return gates, p


@functools.lru_cache(maxsize=256)
def _terms(ham, n, terms):
    """(coefficients, X masks, Z masks): the periodic Heisenberg chain, or random Pauli strings of weight
    up to 4 (as fermionic and spin models give), with normal coefficients."""
    coef, xs, zs = [], [], []
    if ham == "heisenberg":
        for i in range(n):
            m = (1 << i) | (1 << ((i + 1) % n))
            for sig in "XYZ":
                coef.append(1.0)
                xs.append(m if sig in "XY" else 0)
                zs.append(m if sig in "YZ" else 0)
    else:
        rng = np.random.default_rng(100 * n + terms)
        for _ in range(terms):
            x = z = 0
            for q in rng.permutation(n)[:int(rng.integers(1, min(4, n) + 1))]:
                letter = int(rng.integers(0, 3))
                x |= (letter < 2) << int(q)
                z |= (letter > 0) << int(q)
            coef.append(float(rng.standard_normal()))
            xs.append(x)
            zs.append(z)
    return coef, xs, zs


@functools.lru_cache(maxsize=64)
def _sizes(ncirc, nmin, nmax, dmin, dmax, sizes):
    rng = np.random.default_rng(sizes)
    ns, ds = rng.integers(nmin, nmax + 1, ncirc), rng.integers(dmin, dmax + 1, ncirc)
    return [(int(n), int(d)) for n, d in zip(ns, ds)]


def _uneven(case):
    return _sizes(*(case[k] for k in ("ncirc", "nmin", "nmax", "dmin", "dmax", "sizes")))


def _locs(case):
    """Which qubits a transform or a measurement takes, and in which order."""
    n, k = case["n"], case["k"]
    if k == n:
        return list(range(n))
    return [int(q) for q in np.random.default_rng(10 * n + k).permutation(n)[:k]]


def _instructions(n):
    """(kind, target, controls, angle) on the second qubit and on the highest one."""
    return [("X", 1, (), 0.0), ("H", 1, (), 0.0), ("T", 1, (), 0.0), ("Rx", n - 1, (), 0.3), ("X", 1, (2,), 0.0),
            ("X", 1, (2, 3), 0.0)]


# ---- handles that a program keeps -------------------------------------------------------------


@functools.lru_cache(maxsize=1)
def _library():
    yb.init()
    yb.use_torch_stream()


@functools.lru_cache(maxsize=128)
def _circuit(circ, n, depth):
    gates, _ = _gates(circ, n, depth)
    c = yb.Circuit(n)
    for kind, q, ctrls, param, G in gates:
        c.push(kind, (q,), param=param, G=G, ctrls=ctrls)
    return c


@functools.lru_cache(maxsize=128)
def _hamiltonian(ham, n, terms):
    coef, xs, zs = _terms(ham, n, terms)
    return yb.PauliSum(n, coef, np.array(xs, np.uint64), np.array(zs, np.uint64))


@functools.lru_cache(maxsize=4)
def _uneven_handles(sizes, dtype):
    states = [yb.State(n, 1, DTYPES[dtype][0]) for n, _ in sizes]
    circs = [_circuit("hea", n, d) for n, d in sizes]
    return states, circs, [_hamiltonian("heisenberg", n, 0) for n, _ in sizes]


def _angles(seed, count):
    return np.random.default_rng(seed).uniform(0.0, 2.0 * math.pi, count)


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _random_state(case, seed):
    """A normalised complex Gaussian state in every slot."""
    ct = DTYPES[case["dtype"]][1]
    rt = torch.float32 if ct == torch.complex64 else torch.float64
    g = torch.Generator(device=_device()).manual_seed(seed)
    psi = torch.randn((1 << case["n"], case["batch"], 2), dtype=rt, device=_device(), generator=g)
    psi /= psi.double().square().sum((0, 2), keepdim=True).sqrt().to(rt)
    return torch.view_as_complex(psi)


def prepare(case, seed):
    _library()
    kind = case["kind"]
    if kind == "uneven":
        sizes = tuple(_uneven(case))
        states, circs, hams = _uneven_handles(sizes, case["dtype"])
        return dict(case=case, states=states, circs=circs, hams=hams,
                    params=[_angles([seed, c], 3 * n * d) for c, (n, d) in enumerate(sizes)])
    n, dt = case["n"], DTYPES[case["dtype"]]
    s = dict(case=case)
    if kind in ("vqe", "forward", "shift"):
        circ = case.get("circ", "hea")
        s["circ"] = _circuit(circ, n, case["depth"])
        s["params"] = _angles(seed, s["circ"].nparams)
        if kind != "forward":
            s["ham"] = _hamiltonian("heisenberg", n, 0)
    elif kind in ("energy", "evolve"):
        s["ham"] = _hamiltonian(case["ham"], n, case["terms"])
    elif kind == "measure":
        s["u"] = np.random.default_rng(seed).random((case["batch"], case["shots"]))
    if kind == "vqe" or case.get("circ") == "hea":
        s["tensor"] = torch.empty((1 << n, case["batch"]), dtype=dt[1], device="cuda")
        if case["batch"] > 1:
            s["input"] = _random_state(case, seed)
    else:
        s["tensor"] = _random_state(case, seed)
    s["state"] = yb.State(n, case["batch"], dt[0], tensor=s["tensor"])
    if kind == "energy" and case["hpsi"]:
        s["out"] = torch.empty_like(s["tensor"])
        s["out_state"] = yb.State(n, case["batch"], dt[0], tensor=s["out"])
    return s


def run(s):
    case = s["case"]
    kind, single = case["kind"], case["dtype"] == "c64"
    if kind == "uneven":
        e, g = yb.batch_run(s["states"], s["circs"], s["params"], s["hams"])
        g = np.concatenate(g)
        return {"energy": e.astype(np.float32) if single else e, "grad": g.astype(np.float32) if single else g}
    state = s["state"]
    if kind == "vqe":
        if case["batch"] > 1:
            s["tensor"].copy_(s["input"])
        else:
            state.reset()
        e, g, _ = yb.backward(state, s["circ"], s["params"], s["ham"])
        eg = np.concatenate((e[:, None], g), axis=1)  # value and gradient of each slot, as an optimiser takes them
        return {"energy_grad": eg.astype(np.float32) if single else eg, "state": s["tensor"]}
    if kind == "shift":
        e, g = yb.shift_grad(state, s["circ"], s["params"], s["ham"])
        eg = np.concatenate(([e], g))
        return {"energy_grad": eg.astype(np.float32) if single else eg}
    if kind == "forward":
        if case["circ"] == "hea":
            state.reset()
        yb.forward(state, s["circ"], s["params"])
    elif kind == "instr":
        for name, q, ctrls, theta in _instructions(case["n"]):
            state.apply_gate(name, (q,), theta=theta, ctrls=ctrls)
    elif kind == "energy":
        if case["hpsi"]:
            e = yb.hpsi(state, s["ham"], s["out_state"])
            return {"energy": e.astype(np.float32) if single else e, "hpsi": s["out"]}
        e = yb.expect(state, s["ham"])
        return {"energy": e.astype(np.float32) if single else e}
    elif kind == "evolve":
        yb.time_evolve(state, s["ham"], case["t"])
    elif kind == "qft":
        locs = _locs(case)
        if case["focus"]:
            yb.focus(state, locs)
            yb.qft(state, list(range(case["k"])), case["inverse"])
            yb.relax(state, locs)
        else:
            yb.qft(state, locs, case["inverse"])
    elif kind == "measure":
        return {"outcomes": yb.measure(state, _locs(case), s["u"])}
    return {"state": s["tensor"]}


# ---- what a pass cannot do without -------------------------------------------------------------

# Real operations per amplitude: a rotation about X or Z 6, a dense 2x2 14, a swap none.
GATE_FLOPS = {"Rx": 6, "Rz": 6, "dense": 14, "H": 6, "T": 3, "X": 0, "Z": 1}


def _sweep_flops(circ, n, depth):
    return sum(GATE_FLOPS[k] * 2.0 ** (n - len(c)) for k, _, c, _, _ in _gates(circ, n, depth)[0])


def _vqe_flops(n, depth):
    # Forward, psi and lambda back, 4 a gradient and amplitude, and 6 an observable's term and amplitude.
    return 3 * _sweep_flops("hea", n, depth) + (3 * n * depth * 4 + 3 * n * 6) * 2.0 ** n


def work(case):
    kind, b = case["kind"], DTYPES[case["dtype"]][2]
    if kind == "uneven":
        sizes = _uneven(case)
        return {"bytes": sum(b * 2.0 ** n + 16 * 3 * n * d for n, d in sizes), "flops": sum(_vqe_flops(n, d) for n, d in sizes)}
    n, B = case["n"], case["batch"]
    state = b * 2.0 ** n * B
    if kind == "vqe":
        return {"bytes": state + 8 * 3 * n * case["depth"] * (1 + B), "flops": _vqe_flops(n, case["depth"]) * B}
    if kind == "shift":
        circuits = 2 * 3 * n * case["depth"] + 1
        return {"bytes": state + 16 * 3 * n * case["depth"],
                "flops": circuits * (_sweep_flops("hea", n, case["depth"]) + 18.0 * n * 2 ** n)}
    if kind == "forward":
        return {"bytes": 2 * state, "flops": _sweep_flops(case["circ"], n, case["depth"])}
    if kind == "instr":
        moved = [2.0 ** (1 - len(c)) * (0.5 if k == "T" else 1.0) for k, _, c, _ in _instructions(n)]
        return {"bytes": state * sum(moved), "flops": sum(GATE_FLOPS[k] * 2.0 ** (n - len(c)) * B for k, _, c, _ in _instructions(n))}
    if kind in ("energy", "evolve"):
        apply_h = 6.0 * len(_terms(case["ham"], n, case["terms"])[0]) * 2 ** n * B
        if kind == "energy":
            return {"bytes": state * (2 if case["hpsi"] else 1), "flops": apply_h}
        return {"bytes": 2 * state, "flops": 30 * apply_h}
    if kind == "qft":
        return {"bytes": 2 * state, "flops": 5.0 * case["k"] * 2 ** n * B}
    return {"bytes": state + 16.0 * case["shots"] * B, "flops": 4.0 * 2 ** n * B}


# ---- the same in 64 bits ------------------------------------------------------------------------

_R = math.sqrt(0.5)
_FIXED = {"X": [[0, 1], [1, 0]], "Z": [[1, 0], [0, -1]], "H": [[_R, _R], [_R, -_R]], "T": [[1, 0], [0, complex(_R, _R)]]}


def _matrix(kind, theta, G):
    if kind == "dense":
        return G
    if kind == "Rx":
        c, s = math.cos(theta / 2), math.sin(theta / 2)
        return [[c, -1j * s], [-1j * s, c]]
    if kind == "Rz":
        return [[complex(math.cos(theta / 2), -math.sin(theta / 2)), 0], [0, complex(math.cos(theta / 2), math.sin(theta / 2))]]
    return _FIXED[kind]


def _halves(psi, q, ctrls):
    """The amplitudes with qubit q at 0 and at 1 and every control at 1, as views of psi [2^n, B]."""
    cuts = sorted((q,) + tuple(ctrls), reverse=True)
    dims, top = [], psi.shape[0].bit_length() - 1
    for c in cuts:
        dims += [1 << (top - c - 1), 2]
        top = c
    v = psi.view(dims + [1 << top, psi.shape[1]])
    at = [slice(None)] * v.dim()
    for i, c in enumerate(cuts):
        if c != q:
            at[2 * i + 1] = 1
    t = 2 * cuts.index(q) + 1
    a, b = list(at), list(at)
    a[t], b[t] = 0, 1
    return v[tuple(a)], v[tuple(b)]


def _apply(psi, U, q, ctrls=()):
    a, b = _halves(psi, q, ctrls)
    (u00, u01), (u10, u11) = U
    if u01 == 0 and u10 == 0:
        if u00 != 1:
            a.mul_(u00)
        b.mul_(u11)
        return
    old = a.clone()
    a.mul_(u00).add_(b, alpha=u01)
    b.mul_(u11).add_(old, alpha=u10)


def _dagger(U):
    return [[complex(U[j][i]).conjugate() for j in range(2)] for i in range(2)]


def _hpsi(psi, coef, xs, zs):
    out = torch.zeros_like(psi)
    j = torch.arange(psi.shape[0], device=psi.device)
    for c, x, z in zip(coef, xs, zs):
        k = j ^ x
        parity = k & z
        for sh in (16, 8, 4, 2, 1):
            parity ^= parity >> sh
        f = (1 - 2 * (parity & 1)).to(torch.float64).unsqueeze(1)
        out += (c * 1j ** bin(x & z).count("1")) * (f * psi[k])
    return out


def _slots(a, b):
    return (a.conj() * b).sum(tuple(range(a.dim() - 1)))


def _gradient(gates, nparams, angles, psi, terms):
    """(energies [B], gradients [B, nparams], the output state) by the adjoint method; psi is the input."""
    mats = [_matrix(k, angles[p] if p >= 0 else 0.0, G) for k, _, _, p, G in gates]
    for (k, q, ctrls, p, G), U in zip(gates, mats):
        _apply(psi, U, q, ctrls)
    last = psi.clone()
    lam = _hpsi(psi, *terms)
    e = _slots(psi, lam).real
    g = [None] * nparams
    for (k, q, ctrls, p, G), U in zip(reversed(gates), reversed(mats)):
        if p >= 0:
            (la, lb), (a, b) = _halves(lam, q, ctrls), _halves(psi, q, ctrls)
            g[p] = (_slots(la, b) + _slots(lb, a) if k == "Rx" else _slots(la, a) - _slots(lb, b)).imag
        _apply(psi, _dagger(U), q, ctrls)
        _apply(lam, _dagger(U), q, ctrls)
    return e, torch.stack(g, 1), last


def _zero_state(n, batch):
    psi = torch.zeros((1 << n, batch), dtype=torch.complex128, device=_device())
    psi[0] = 1
    return psi


def _shift_gradient(gates, nparams, angles, psi, terms):
    """Every derivative by shifting its angle by half a turn's quarter each way, the shifted circuits side by side."""
    shifts = np.zeros((2 * nparams + 1, nparams))
    for p in range(nparams):
        shifts[2 * p, p], shifts[2 * p + 1, p] = math.pi / 2, -math.pi / 2
    theta = torch.as_tensor(shifts + np.asarray(angles)[None, :], device=psi.device)
    psi = psi.repeat(1, 2 * nparams + 1)
    for k, q, ctrls, p, G in gates:
        if p < 0:
            _apply(psi, _matrix(k, 0.0, G), q, ctrls)
            continue
        c, s = torch.cos(theta[:, p] / 2), torch.sin(theta[:, p] / 2)
        a, b = _halves(psi, q, ctrls)
        if k == "Rx":
            old = a.clone()
            a.mul_(c).add_(-1j * s * b)
            b.mul_(c).add_(-1j * s * old)
        else:
            a.mul_(torch.complex(c, -s))
            b.mul_(torch.complex(c, s))
    e = _slots(psi, _hpsi(psi, *terms)).real
    return torch.cat((e[-1:], (e[0:-1:2] - e[1:-1:2]) / 2))


def _places(n, places, dev):
    """Index i's bit j put at bit places[j]."""
    i = torch.arange(1 << n, device=dev)
    out = torch.zeros_like(i)
    for j, q in enumerate(places):
        out |= ((i >> j) & 1) << q
    return out


def _fourier(psi, locs, inverse):
    """out[y] = 2^{-k/2} sum_x exp(2 pi i rev(x) y / 2^k) psi[x] over the qubits locs, locs[j] bit j of x and y;
    inverse: its adjoint."""
    n, k = psi.shape[0].bit_length() - 1, len(locs)
    rest = [q for q in range(n) if q not in locs]
    plain = _places(n, list(locs) + rest, psi.device)
    reverse = _places(n, list(reversed(locs)) + rest, psi.device)
    out = torch.empty_like(psi)
    if not inverse:
        out[plain, 0] = torch.fft.ifft(psi[reverse, 0].view(-1, 1 << k), norm="ortho").view(-1)
    else:
        out[reverse, 0] = torch.fft.fft(psi[plain, 0].view(-1, 1 << k), norm="ortho").view(-1)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "uneven":
        es, gs = [], []
        for c, (n, d) in enumerate(_uneven(case)):
            gates, p = _gates("hea", n, d)
            e, g, _ = _gradient(gates, p, _angles([seed, c], p), _zero_state(n, 1), _terms("heisenberg", n, 0))
            es.append(e)
            gs.append(g.reshape(-1))
        return {"energy": torch.cat(es), "grad": torch.cat(gs)}
    if kind == "measure":
        return None
    n = case["n"]
    if kind == "vqe":
        gates, p = _gates("hea", n, case["depth"])
        psi = _random_state(case, seed).to(torch.complex128) if case["batch"] > 1 else _zero_state(n, 1)
        e, g, last = _gradient(gates, p, _angles(seed, p), psi, _terms("heisenberg", n, 0))
        return {"energy_grad": torch.cat((e.unsqueeze(1), g), 1), "state": last}
    psi = _random_state(case, seed).to(torch.complex128)
    if kind == "shift":
        gates, p = _gates("hea", n, case["depth"])
        return {"energy_grad": _shift_gradient(gates, p, _angles(seed, p), psi, _terms("heisenberg", n, 0))}
    if kind == "forward":
        gates, p = _gates(case["circ"], n, case["depth"])
        angles = _angles(seed, p)
        if case["circ"] == "hea":
            psi = _zero_state(n, 1)
        for k, q, ctrls, at, G in gates:
            _apply(psi, _matrix(k, angles[at] if at >= 0 else 0.0, G), q, ctrls)
        return {"state": psi}
    if kind == "instr":
        for k, q, ctrls, theta in _instructions(n):
            _apply(psi, _matrix(k, theta, None), q, ctrls)
        return {"state": psi}
    if kind == "qft":
        return {"state": _fourier(psi, _locs(case), case["inverse"])}
    terms = _terms(case["ham"], n, case["terms"])
    if kind == "energy":
        h = _hpsi(psi, *terms)
        e = _slots(psi, h).real
        return {"energy": e, "hpsi": h} if case["hpsi"] else {"energy": e}
    steps = max(1, math.ceil(sum(abs(c) for c in terms[0]) * case["t"] / 4))  # evolve: the exponential's series
    for _ in range(steps):
        term = psi.clone()
        for m in range(1, 41):
            term = _hpsi(term, *terms) * (-1j * case["t"] / steps / m)
            psi = psi + term
    return {"state": psi}
