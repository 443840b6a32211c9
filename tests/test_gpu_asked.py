"""What a run is asked for (probabilities, registers) changes none of its bits:
d <= 3 runs take one kernel whatever is asked for (two that round differently
gave other final bits in two and three of 2e6 complex64 trajectories)."""
import numpy as np
import pytest

import paper_2204_11404_amd as qs

pytestmark = pytest.mark.gpu


# complex64 outcomes whose probability depends on rounding (some 1e-7 wide):
# 2e6 x 32 decisions with probabilities spread over (0, 1) hold several
@pytest.mark.parametrize("zeta", [0.0, 0.01])
def test_probabilities_change_no_outcome(zeta):
    print(f"case asked zeta={zeta}", flush=True)
    kw = dict(d=3, gateset="cr", rounds=4, n_traj=2_000_000, seed=11, p=0.01, eps=0.35, zeta=zeta, dtype="c64")
    a, b = qs.run_rounds(**kw), qs.run_rounds(want_p1=True, **kw)
    assert 0.2 < np.mean((b["p1"][:1000] > 0.02) & (b["p1"][:1000] < 0.98))
    assert np.count_nonzero((a["records"] != b["records"]).any(axis=(1, 2))) == 0
    assert np.array_equal(a["final_bits"], b["final_bits"])


# p = 0.2: Paulis in every round turn both frames and the sign; registers and
# probabilities against the register passes.  Three rounds of 8 checks, about
# ten roundings an amplitude each: 240 half units, twice that in a probability.
@pytest.mark.parametrize("dtype,tol", [("c128", 480 * 2.0**-53), ("c64", 480 * 2.0**-24)])
@pytest.mark.parametrize("d,gateset", [(2, "cr"), (3, "cr"), (3, "textbook")])
@pytest.mark.parametrize("zeta", [0.0, 0.02])
def test_frames_and_sign(monkeypatch, d, gateset, zeta, dtype, tol):
    kw = dict(d=d, gateset=gateset, rounds=3, n_traj=60, seed=23, p=0.2, eps=0.05, zeta=zeta, dtype=dtype, traj0=9,
              want_p1=True)
    monkeypatch.setenv("QECSV_SPEC", "0")
    want = qs.run_rounds(want_states=True, **kw)
    monkeypatch.delenv("QECSV_SPEC")
    got, p1 = qs.run_rounds(want_states=True, **kw), qs.run_rounds(**kw)
    assert np.array_equal(got["records"], want["records"])
    assert np.array_equal(got["final_bits"], want["final_bits"])
    assert np.abs(got["p1"] - want["p1"]).max() <= tol
    assert np.abs(got["states"] - want["states"]).max() <= tol
    assert np.array_equal(p1["p1"], got["p1"])


def test_registers_change_no_final_bit_d5():
    """complex64 d = 5: over-rotations around the value at which a bit of the
    final measurement turns, in steps of the register's rounding."""
    sites = qs.template_info(5, "cr")[1]
    pattern = np.random.default_rng(3).uniform(0.5, 1.0, sites)

    def bits(a, seed, **kw):
        g = qs.run_rounds(d=5, gateset="cr", rounds=1, n_traj=1, seed=seed, p=0.0, eps_site=a * pattern, dtype="c64",
                          **kw)
        return np.concatenate([g["records"].reshape(-1), g["final_bits"].reshape(-1)])

    turned = 0
    for seed in range(16):  # (few seeds have a bit that turns while no outcome does)
        grid = np.linspace(0.05, 0.25, 30)
        rows = [bits(a, seed) for a in grid]
        at = [i for i in range(29) if np.array_equal(rows[i][:24], rows[i + 1][:24]) and
              not np.array_equal(rows[i], rows[i + 1])]
        if not at:
            continue
        lo, hi = grid[at[0]], grid[at[0] + 1]
        while hi - lo > 1e-9 * lo:
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if np.array_equal(bits(mid, seed), rows[at[0]]) else (lo, mid)
        near = lo * (1.0 + np.linspace(-2e-7, 2e-7, 17))
        plain = [bits(a, seed) for a in near]
        turned += len(np.unique(plain, axis=0)) > 1
        print(f"case final bits seed {seed}", flush=True)
        for a, want in zip(near, plain):
            assert np.array_equal(bits(a, seed, want_states=True), want), (seed, a)
    assert turned >= 2
