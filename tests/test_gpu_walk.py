"""Whole-register operations in both directions, and the fused matrices that
move two groups a lane (complex64, bit 0 no target)."""
import numpy as np
import pytest

import paper_2204_11404_amd as qs
import workloads
from oracle import statevec as sv

pytestmark = pytest.mark.gpu


def _unitary(k, rng):
    a = rng.normal(size=(1 << k, 1 << k)) + 1j * rng.normal(size=(1 << k, 1 << k))
    return np.linalg.qr(a)[0]


# One B tile pair (n - k = 5), several a wave, a remainder of waves; targets at
# both ends, unsorted, next to bit 0 and without it.  Three unitaries in a row,
# sums of 32 complex terms on vectors of norm 1 at most: 3 * 130 half units.
@pytest.mark.parametrize("dtype,tol", [("c128", 400 * 2.0**-53), ("c64", 400 * 2.0**-24)])
@pytest.mark.parametrize("n,qubits", [(9, [1, 2, 3, 4]), (9, [8, 1, 5, 3]), (10, [1, 2, 3, 4, 5]),
                                      (10, [9, 7, 1, 3, 2]), (10, [9, 7, 0, 3, 2]), (13, [12, 1, 11, 2, 6]),
                                      (14, [13, 12, 11, 10]), (15, [4, 3, 2, 1, 0])])
def test_fused_both_directions(dtype, tol, n, qubits):
    k = len(qubits)
    psi = workloads.random_state(n, n + k)
    s = qs.State(n, dtype)
    s.set(psi)
    ref = s.get().astype(np.complex128)
    for i in range(3):
        m = _unitary(k, np.random.default_rng(31 * n + i))
        s.apply_fused(qubits, m)
        ref = sv.apply_gate(ref, qubits, m)
    assert np.max(np.abs(s.get() - ref)) < tol
    s.free()


@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 2e-5)])
@pytest.mark.parametrize("n", [1, 2, 8, 10, 13])
def test_sequence_of_operations(dtype, tol, n):
    """Gates, phases and measurements in turn, each walking the other way."""
    psi = workloads.random_state(n, 3 * n)
    s = qs.State(n, dtype)
    s.set(psi)
    ref = s.get().astype(np.complex128)
    rng = np.random.default_rng(n)

    for i in range(7):
        k = 1 + (i & 1) if n > 1 else 1
        qubits = list(rng.permutation(n)[:k])
        m = _unitary(k, rng)
        s.apply_gate([int(q) for q in qubits], m)
        ref = sv.apply_gate(ref, qubits, m)
        ph = np.exp(1j * rng.uniform(0, 6, 2))
        q = int(rng.integers(n))
        s.apply_diag([q], ph)
        ref = sv.apply_gate(ref, [q], np.diag(ph))
        if i in (2, 5):
            bit = (np.arange(1 << n) >> q) & 1
            p1 = float(np.sum(np.abs(ref[bit == 1]) ** 2) / np.sum(np.abs(ref) ** 2))
            m1, got = s.measure_reset(q, 0.5)
            assert abs(got - p1) < tol and m1 == (1 if 0.5 < p1 else 0)
            kept = ref[bit == m1] / np.sqrt(np.sum(np.abs(ref[bit == m1]) ** 2))
            ref = np.zeros_like(ref)
            ref[bit == 0] = kept
    assert np.max(np.abs(s.get() - ref)) < tol
    s.free()
