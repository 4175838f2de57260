"""H psi and energies over the register sizes where the observable kernels change: the one-launch form
with two elements a thread (up to 17 qubits), four (up to 20, and above for few X masks), tile passes,
and X masks wider than a tile; with Y letters and Z letters on every index bit.

The input is the state as the register holds it, so only the sums round: with S = sum |c|, FP64 sums of a
few dozen terms stay within 1e-12 S (times the largest amplitude for H psi), and a complex64 output
adds its rounding, 6e-8 of a value of at most S times the largest amplitude, per pass."""
import numpy as np
import pytest

import oracle
import workloads as w

pytestmark = pytest.mark.gpu


def pauli_strings(n, seed, wide):
    """Random strings of every weight on random qubits, each top qubit in X, Y and Z once, two strings that
    share an X mask with different letters, a constant, and a mask of 14 X letters if wide."""
    rng = np.random.default_rng(seed)
    strings = ["I" * n]
    for weight in (1, 2, 3, min(4, n)):
        for _ in range(3):
            s = ["I"] * n
            for q in rng.permutation(n)[:weight]:
                s[q] = "XYZ"[int(rng.integers(3))]
            strings.append("".join(s))
    for q in range(n - 4, n):
        strings += ["I" * q + p + "I" * (n - q - 1) for p in "XYZ"]
    strings += ["XX" + "I" * (n - 2), "YY" + "I" * (n - 2), "I" * (n - 2) + "YX", "I" * (n - 2) + "XY"]
    if wide:
        strings.append("X" * 13 + "Y" + "I" * (n - 14))
    return w.pauli_sum(n, [(float(c), s) for c, s in zip(rng.standard_normal(len(strings)), strings)])


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n,B,wide", [(4, 1, False), (5, 1, False), (8, 1, False), (9, 1, False), (9, 3, False), (17, 1, False),
                                      (18, 1, True), (20, 1, False), (21, 1, False), (21, 1, True), (14, 2, True)])
def test_observable_forms(dtype, n, B, wide):
    from paper_1912_10877_amd import binding as yb

    yb.init()
    H = pauli_strings(n, 31 + n, wide)
    s, out = yb.State(n, B, dtype), yb.State(n, B, dtype)
    s.upload(w.random_state(n, B, n))
    psi = s.download().astype(np.complex128)
    ref = oracle.hpsi(H, psi).reshape(psi.shape)
    e_ref = np.sum(psi.conj() * ref, axis=0).real
    h = yb.PauliSum.from_workload(H)
    total, top = float(np.abs(H.coef).sum()), float(np.abs(psi).max())
    e = yb.hpsi(s, h, out)
    tol = (1e-12 if dtype == 1 else 4 * 6e-8) * total * top
    assert np.abs(out.download() - ref).max() <= tol
    assert np.abs(e - e_ref).max() <= 1e-12 * total
    assert np.abs(yb.expect(s, h) - e_ref).max() <= 1e-12 * total


def test_energy_of_many_tiles():
    """Enough tiles that the partial sums of a slot take the workgroup-wide sum: |+> on 23 qubits."""
    from paper_1912_10877_amd import binding as yb

    yb.init()
    n = 23
    s = yb.State(n, 1, 0)
    s.upload(np.full(1 << n, 2.0 ** (-n / 2), np.complex128))
    e = yb.expect(s, yb.PauliSum.from_workload(w.heisenberg(n)))  # XX of every bond
    assert abs(e[0] - n) <= 1e-6 * n  # the amplitude's float rounding, squared


def low_masks(n, nterms, seed):
    """Random strings on n qubits whose X masks lie on the 12 lowest, one pass over tiles."""
    rng = np.random.default_rng(seed)
    xs, zs = rng.integers(1, 1 << 12, nterms), rng.integers(0, 1 << n, nterms)
    strings = ["".join("IXZY"[int(x >> q & 1) + 2 * int(z >> q & 1)] for q in range(n)) for x, z in zip(xs, zs)]
    return w.pauli_sum(n, [(float(c), s) for c, s in zip(rng.standard_normal(nterms), strings)])


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [18, 20, 21])
def test_many_masks_in_one_tile(n, dtype):
    """A hundred X masks in one tile, where single-slot states of 18 to 20 qubits take tile passes: H psi and the
    energy to the bounds above, and a short evolution (its Krylov steps in separate launches) to the bounds
    of the evolution tests, 1e-10 and 2e-5 an amplitude."""
    from paper_1912_10877_amd import binding as yb

    yb.init()
    H = low_masks(n, 100, 77)
    s, out = yb.State(n, 1, dtype), yb.State(n, 1, dtype)
    s.upload(w.random_state(n, 1, n))
    psi = s.download().astype(np.complex128)
    ref = oracle.hpsi(H, psi).reshape(psi.shape)
    e_ref = np.sum(psi.conj() * ref, axis=0).real
    h = yb.PauliSum.from_workload(H)
    total, top = float(np.abs(H.coef).sum()), float(np.abs(psi).max())
    e = yb.hpsi(s, h, out)
    assert np.abs(out.download() - ref).max() <= (1e-12 if dtype == 1 else 4 * 6e-8) * total * top
    assert np.abs(e - e_ref).max() <= 1e-12 * total
    assert np.abs(yb.expect(s, h) - e_ref).max() <= 1e-12 * total
    if n == 18:
        steps = yb.time_evolve(s, h, 0.02)
        assert np.abs(s.download() - oracle.time_evolve(H, psi, 0.02)).max() <= (1e-10 if dtype == 1 else 2e-5) * steps


def test_energies_of_one_state_cost_no_more_than_of_two():
    """400 X masks in one tile, 20 qubits complex128: a batch of two states always takes the tile passes, so one
    state must not take longer, whichever form is chosen for it (the gathering launch takes five times
    as long here)."""
    import time

    from paper_1912_10877_amd import binding as yb

    yb.init()
    n = 20
    h = yb.PauliSum.from_workload(low_masks(n, 400, 78))
    us = []
    for B in (1, 2):
        s, out = yb.State(n, B, 1), yb.State(n, B, 1)
        for call in (lambda: yb.expect(s, h), lambda: yb.hpsi(s, h, out)):
            call()
            took = []
            for _ in range(15):
                t0 = time.perf_counter()
                call()
                took.append(time.perf_counter() - t0)
            us.append(1e6 * float(np.median(took)))
    assert us[0] <= us[2] and us[1] <= us[3], us


def test_tables_of_many_terms():
    """The launch tables of an observable are made on its first energy and, for H psi, once more: with 20000 terms
    of nearly as many X masks both take a fraction of the time that making the observable takes (which
    looks for every mask among all others)."""
    import time

    from paper_1912_10877_amd import binding as yb

    yb.init()
    n, k = 20, 20000
    rng = np.random.default_rng(79)
    x, z, c = rng.integers(0, 1 << n, k).astype(np.uint64), rng.integers(0, 1 << n, k).astype(np.uint64), rng.standard_normal(k)
    s, out = yb.State(n, 1, 1), yb.State(n, 1, 1)
    small = yb.PauliSum(n, c[:3], x[:3], z[:3])
    yb.expect(s, small), yb.hpsi(s, small, out)
    t = [time.perf_counter()]
    h = yb.PauliSum(n, c, x, z)
    t.append(time.perf_counter())
    for call in (lambda: yb.expect(s, h), lambda: yb.hpsi(s, h, out)) * 2:
        call()
        t.append(time.perf_counter())
    made, first_e, first_v, again_e, again_v = np.diff(t)
    assert first_e - again_e <= 0.5 * made and first_v - again_v <= 0.5 * made, np.diff(t)
