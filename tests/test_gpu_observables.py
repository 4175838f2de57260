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
