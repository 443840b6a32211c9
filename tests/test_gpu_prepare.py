"""Kraus pairs of a run: every trajectory and round of a check, in groups of
four a wave with remainders, as when it runs alone."""
import numpy as np
import pytest

import paper_2204_11404_amd as qs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_traj,rounds", [(1, 1), (1, 3), (2, 2), (3, 3), (5, 1)])
@pytest.mark.parametrize("d,gateset,flag", [(3, "cr", "xbasis"), (3, "cr", "idle_noise"), (3, "textbook", "twirl"),
                                            (2, "cr", "zz_plaquette"), (4, "cr", None)])
def test_groups_and_remainders(d, gateset, flag, n_traj, rounds):
    kw = dict(d=d, gateset=gateset, rounds=rounds, seed=77, p=0.3, eps=0.04, dtype="c128", zeta=0.02, want_p1=True)
    if flag:
        kw[flag] = True
    whole = qs.run_rounds(n_traj=n_traj, traj0=2, **kw)
    for t in range(n_traj):
        one = qs.run_rounds(n_traj=1, traj0=2 + t, **kw)
        assert np.array_equal(one["records"][0], whole["records"][t])
        assert np.array_equal(one["final_bits"][0], whole["final_bits"][t])
        # (a register's sums may be split differently: two roundings a sum)
        assert np.abs(one["p1"][0] - whole["p1"][t]).max() <= 1e-12


@pytest.mark.parametrize("n", [1, 3, 6])
def test_batch_slots_match_single_runs(n):
    n_sites = qs.template_info(4, "cr")[1]
    rng = np.random.default_rng(n)
    rounds, p = rng.integers(1, 4, n), rng.uniform(0.1, 0.3, n)
    eps = rng.normal(0.0, 0.03, (n, n_sites))
    out = qs.run_batch(4, "cr", rounds, p, 9, eps_site=eps, dtype="c128", max_rounds=3, zeta=0.01)
    for t in range(n):
        one = qs.run_rounds(d=4, gateset="cr", rounds=int(rounds[t]), n_traj=1, traj0=t, seed=9, p=float(p[t]),
                            eps_site=eps[t], dtype="c128", zeta=0.01)
        assert np.array_equal(out["records"][t, : rounds[t]], one["records"][0])
        assert np.array_equal(out["final_bits"][t], one["final_bits"][0])
