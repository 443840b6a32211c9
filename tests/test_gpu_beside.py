"""A d = 4 batched trajectory's bits do not depend on how many run beside it.

Over-rotations next to the value at which an outcome turns: its probability
there is its draw to the last bit, so sums added in another order turn it at
another value."""
import numpy as np
import pytest

import paper_2204_11404_amd as qs

pytestmark = pytest.mark.gpu

ROUNDS = 2


def _records(scales, n, dtype, seed):
    """Records of a trajectory (draw stream 0, noise-free, one angle pattern
    times each of `scales`) that is the first of a batch of n."""
    sites = qs.template_info(4, "cr")[1]
    pattern = np.random.default_rng(5).uniform(0.5, 1.0, sites)
    out = []
    for a in scales:
        eps = np.full((n, sites), 0.1)
        eps[0] = a * pattern
        out.append(qs.run_batch(4, "cr", np.full(n, ROUNDS, np.int32), np.zeros(n), seed, dtype=dtype,
                                max_rounds=ROUNDS, eps_site=eps)["records"][0].reshape(-1))
    return np.stack(out)


def turning_point(f, lo, hi, left):
    """The last double in [lo, hi] at which f is still `left`."""
    while True:
        mid = 0.5 * (lo + hi)
        if mid in (lo, hi):
            return lo
        lo, hi = (mid, hi) if np.array_equal(f(mid), left) else (lo, mid)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_batch_of_any_size(dtype):
    """Alone (as many workgroups as tiles) and beside 49, 99 and 399 others
    (down to four tiles each), at turning points of checks after the first
    chain, whose sums are those of the initial state's equal amplitudes."""
    print(f"case beside {dtype}", flush=True)
    points = 0
    for seed in range(8):
        grid = np.linspace(0.02, 0.6, 40)
        rows = _records(grid, 1, dtype, seed)
        at = [i for i in range(len(grid) - 1)
              if np.array_equal(rows[i][:8], rows[i + 1][:8]) and not np.array_equal(rows[i], rows[i + 1])]
        for i in at[:2]:
            t = turning_point(lambda a: _records([a], 1, dtype, seed)[0], grid[i], grid[i + 1], rows[i])
            near = t + np.spacing(t) * np.arange(-16, 17)
            alone = _records(near, 1, dtype, seed)
            points += len(np.unique(alone, axis=0)) > 1
            for n in (50, 100, 400):
                assert np.array_equal(_records(near, n, dtype, seed), alone), (seed, i, n)
    assert points >= 4
