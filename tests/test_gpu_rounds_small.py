"""d <= 3 runs as one on-chip launch against the passes (QECSV_SPEC = 0)."""
import numpy as np
import pytest

import paper_2204_11404_amd as qs

pytestmark = pytest.mark.gpu


def _run(monkeypatch, passes, **kw):
    if passes:
        monkeypatch.setenv("QECSV_SPEC", "0")
    else:
        monkeypatch.delenv("QECSV_SPEC", raising=False)
    return qs.run_rounds(**kw)


# Up to 3 rounds of 8 checks, about ten roundings an amplitude each: relative
# errors of 240 half units, twice that in a probability.
@pytest.mark.parametrize("dtype,tol", [("c128", 480 * 2.0**-53), ("c64", 480 * 2.0**-24)])
@pytest.mark.parametrize("d,gateset,n_traj,rounds", [(2, "cr", 1, 3), (3, "cr", 1, 1), (3, "textbook", 7, 3),
                                                     (3, "cr", 40, 3)])
@pytest.mark.parametrize("zeta,virtual_z", [(0.0, False), (0.01, False), (0.01, True)])
def test_small_run_matches_passes(monkeypatch, d, gateset, n_traj, rounds, dtype, tol, zeta, virtual_z):
    if virtual_z and gateset != "cr":
        pytest.skip("virtual Z restores belong to the cross-resonance set")
    n_sites = qs.template_info(d, gateset)[1]
    eps = np.random.default_rng(d * 100 + n_traj).normal(0.0, 0.03, n_sites)
    kw = dict(d=d, gateset=gateset, rounds=rounds, n_traj=n_traj, seed=21, p=0.02, eps_site=eps, zeta=zeta,
              dtype=dtype, traj0=5, virtual_z=virtual_z)
    want = _run(monkeypatch, True, want_p1=True, want_states=True, **kw)
    got = _run(monkeypatch, False, want_p1=True, want_states=True, **kw)
    assert got["passes_per_round"] == want["passes_per_round"]
    assert np.array_equal(got["records"], want["records"])
    assert np.array_equal(got["final_bits"], want["final_bits"])
    assert np.abs(got["p1"] - want["p1"]).max() <= tol
    assert np.abs(got["states"] - want["states"]).max() <= tol
    plain = _run(monkeypatch, False, **kw)  # neither asked for
    assert np.array_equal(plain["records"], want["records"])
    assert np.array_equal(plain["final_bits"], want["final_bits"])


def test_small_run_in_several_launches(monkeypatch):
    """Results beyond 256 MiB: 40 000 registers of 8 KiB take two launches."""
    kw = dict(d=3, gateset="cr", rounds=1, seed=3, p=0.01, eps=0.02, dtype="c128", want_states=True)
    whole = _run(monkeypatch, False, n_traj=40000, **kw)
    part = _run(monkeypatch, False, n_traj=2, traj0=39998, **kw)
    assert np.array_equal(whole["records"][-2:], part["records"])
    assert np.array_equal(whole["states"][-2:], part["states"])
