"""Set-up copies and results of a call in one block: sizes on both sides of the
pinned block, without it (no-allocation batches), several threads at once."""
import threading

import numpy as np
import pytest

import paper_2204_11404_amd as qs

pytestmark = pytest.mark.gpu


def _batch(n, no_alloc=False, seed=5):
    ns = qs.template_info(3, "cr")[1]
    rng = np.random.default_rng(n)
    rounds = rng.integers(1, 5, n)
    p = rng.uniform(0.0, 0.02, n)
    eps = rng.normal(0.0, 0.02, (n, ns))
    return qs.run_batch(3, "cr", rounds, p, seed, eps_site=eps, dtype="c64", max_rounds=4, no_alloc=no_alloc)


# 600: angles inside the block's part; 3000: angles apart; 40000: inputs and
# results beyond a pinned block
@pytest.mark.parametrize("n", [1, 600, 3000, 40000])
def test_batch_sizes_match_no_alloc(n):
    a, b = _batch(n), _batch(n, no_alloc=True)
    assert np.array_equal(a["records"], b["records"])
    assert np.array_equal(a["final_bits"], b["final_bits"])


# 4000 x 36 outcomes with their probabilities: beyond a pinned block; 4: within
@pytest.mark.parametrize("n_traj", [4, 4000])
def test_run_rounds_sizes(n_traj):
    kw = dict(d=2, gateset="cr", rounds=12, eps=0.03, p=0.01, seed=9, dtype="c128", want_p1=True)
    whole = qs.run_rounds(n_traj=n_traj, **kw)
    part = qs.run_rounds(n_traj=3, traj0=n_traj - 3, **kw)
    for k in ("records", "final_bits", "p1"):
        assert np.array_equal(whole[k][-3:], part[k]), k


def test_threads_share_the_blocks():
    want = _batch(600)
    got = [None] * 12

    def work(i):
        for _ in range(4):
            got[i] = _batch(600)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(got))]
    [t.start() for t in ts]
    [t.join() for t in ts]
    for g in got:
        assert np.array_equal(g["records"], want["records"])
        assert np.array_equal(g["final_bits"], want["final_bits"])
