"""Operations on registers larger than the last-level cache, which walk in turn
forwards and backwards, and the fused matrices that move two groups a lane with
several tiles a wave, the next one's loads ahead."""
import numpy as np
import pytest

import paper_2204_11404_amd as qs

pytestmark = pytest.mark.gpu


def _unitary(k, rng):
    a = rng.normal(size=(1 << k, 1 << k)) + 1j * rng.normal(size=(1 << k, 1 << k))
    return np.linalg.qr(a)[0]


def _random(n, dtype):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    v = torch.randn((1 << n, 2), generator=g, device="cuda", dtype=torch.float64 if dtype == "c128" else torch.float32)
    return torch.view_as_complex(v / np.sqrt(2.0 * 2.0**n))


def _apply(v, n, qubits, m):
    """m on the given qubits (bit j of its index: qubits[j]) in complex128."""
    import torch
    k = len(qubits)
    axes = [n - 1 - q for q in reversed(qubits)]  # of v as n axes of two, the highest qubit first
    t = torch.movedim(v.reshape((2,) * n), axes, list(range(k)))
    w = torch.as_tensor(m, dtype=torch.complex128, device=v.device) @ t.reshape(1 << k, -1)
    return torch.movedim(w.reshape((2,) * n), list(range(k)), axes).reshape(-1)


# seven operations: sums of at most 32 complex terms each, on vectors of norm 1
@pytest.mark.parametrize("n,dtype,tol", [(25, "c128", 900 * 2.0**-53), (26, "c64", 900 * 2.0**-24),
                                         (24, "c128", 900 * 2.0**-53)])
def test_both_directions(n, dtype, tol):
    """512 MiB, and 256 MiB (one direction)."""
    import torch
    print(f"case large walk {n} {dtype}", flush=True)
    t = _random(n, dtype)
    ref = t.to(torch.complex128, copy=True)
    s = qs.State(n, dtype, stream=torch.cuda.current_stream(), tensor=t)
    rng = np.random.default_rng(n)
    for op, q in (("gate", [n - 1]), ("gate", [3, n - 2]), ("diag", [1, n - 3, 7]), ("gate", [1, 0]),
                  ("fused", [2, 9, n - 1]), ("fused", [n - 4, 5, 1, 12]), ("fused", [4, 0, 1, 3, 2])):
        if op == "diag":
            ph = np.exp(1j * rng.uniform(0, 6, 1 << len(q)))
            s.apply_diag(q, ph)
            ref = _apply(ref, n, q, np.diag(ph))
        else:
            m = _unitary(len(q), rng)
            (s.apply_gate if op == "gate" else s.apply_fused)(q, m)
            ref = _apply(ref, n, q, m)
    m1, p1 = s.measure_reset(n - 2, 0.4)
    w = ref.reshape(2, 2, -1)
    w = w / torch.linalg.vector_norm(w)
    assert abs(p1 - float(torch.linalg.vector_norm(w[:, 1]) ** 2)) < tol and m1 == int(0.4 < p1)
    kept = w[:, m1] / torch.linalg.vector_norm(w[:, m1])
    got = t.reshape(2, 2, -1)
    assert float(torch.abs(got[:, 0] - kept).max()) < tol
    assert float(torch.abs(got[:, 1]).max()) == 0.0


@pytest.mark.parametrize("n,qubits", [(23, [22, 1, 9, 4]), (24, [20, 21, 22, 23]), (24, [5, 1, 17, 23, 2]),
                                      (26, [1, 2, 3, 4, 5])])
def test_fused_several_tiles_a_wave(n, qubits):
    import torch
    print(f"case fused tiles {n} {qubits}", flush=True)
    t = _random(n, "c64")
    ref = t.to(torch.complex128, copy=True)
    s = qs.State(n, "c64", stream=torch.cuda.current_stream(), tensor=t)
    for i in range(2):
        m = _unitary(len(qubits), np.random.default_rng(31 * n + i))
        s.apply_fused(qubits, m)
        ref = _apply(ref, n, qubits, m)
    # two sums of 32 complex terms on a vector of norm 1
    assert float(torch.abs(t - ref).max()) < 270 * 2.0**-24


@pytest.mark.parametrize("n,qubits", [(18, [17, 1, 9, 4]), (19, [1, 18, 9, 4]), (19, [5, 1, 17, 13, 2]),
                                      (20, [1, 2, 3, 4, 19])])
def test_fused_at_the_edge_of_two_groups_a_lane(n, qubits):
    """The largest registers that take one group a lane and the smallest that
    take two: a tile of 32 groups a SIMD on 256 compute units."""
    import torch
    print(f"case fused edge {n} {qubits}", flush=True)
    t = _random(n, "c64")
    ref = t.to(torch.complex128, copy=True)
    s = qs.State(n, "c64", stream=torch.cuda.current_stream(), tensor=t)
    m = _unitary(len(qubits), np.random.default_rng(n))
    s.apply_fused(qubits, m)
    # one sum of at most 32 complex terms on a vector of norm 1
    assert float(torch.abs(t - _apply(ref, n, qubits, m)).max()) < 135 * 2.0**-24
