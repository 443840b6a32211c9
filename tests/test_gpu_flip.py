"""Basis-change passes (sv_run_rounds at d = 5 and sv_run_batch at d = 4
without the data ZZ layer) against the plain passes, which the oracle checks.

The register is kept partly in the Hadamard basis and chains of checks of
either type are summed at once (see k_flip).  Records and final bits must
agree bit for bit with the plain passes (QECSV_SPEC=0); in complex128 p1 and
the register to 1e-12 (some 200 roundings of 1e-16 on each side, amplitudes
and probabilities at most 1), in complex64 to the precision's 1e-5.  p = 0.01
and 0.03 draw Paulis in most rounds, so both frames and the sign are turned.
"""
import numpy as np
import pytest

import paper_2204_11404_amd as qs
import workloads


@pytest.mark.parametrize("gateset", ["cr", "textbook"])
def test_flip_layouts(gateset):
    """Host check of every pass's layouts: five passes a round at d = 5 (44
    basis changes of qubits beside the three lowest, nine a pass), three at
    d = 4, none for registers smaller than a tile."""
    assert [qs.check_flip_layouts(d, gateset) for d in (2, 3, 4, 5)] == [0, 0, 3, 5]


def _both(monkeypatch, run):
    monkeypatch.delenv("QECSV_SPEC", raising=False)
    a = run()
    monkeypatch.setenv("QECSV_SPEC", "0")
    b = run()
    assert np.array_equal(a["records"], b["records"])
    assert np.array_equal(a["final_bits"], b["final_bits"])
    return a, b


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("gateset,flag", [("cr", ""), ("textbook", ""), ("cr", "xbasis"), ("cr", "twirl"),
                                          ("textbook", "idle_noise"), ("cr", "virtual_z")])
def test_flip_matches_plain_passes_d5(monkeypatch, gateset, flag, dtype):
    print(f"case flip d=5 {gateset} {flag} {dtype}", flush=True)
    n_sites = qs.template_info(5, gateset)[1]
    kw = dict(d=5, gateset=gateset, rounds=3, n_traj=2, seed=71, p=0.01, zeta=0.0, dtype=dtype,
              eps_site=workloads.eps_sites(n_sites, (0.0, 0.1), 71), want_p1=True, want_states=True)
    if flag:
        kw[flag] = True
    a, b = _both(monkeypatch, lambda: qs.run_rounds(**kw))
    tol = 1e-12 if dtype == "c128" else 1e-5
    assert a["passes_per_round"] == 5 and a["redo_passes"] == 0
    assert np.max(np.abs(a["p1"] - b["p1"])) < tol
    assert np.max(np.abs(a["states"] - b["states"])) < tol


@pytest.mark.gpu
def test_flip_graph_and_async_d5(monkeypatch):
    """The captured sequence, replayed with an eager run between two graph
    runs, and the enqueued run give the stream launches' results bit for bit."""
    import torch
    monkeypatch.delenv("QECSV_SPEC", raising=False)
    kw = dict(d=5, gateset="cr", rounds=2, n_traj=3, seed=73, p=0.01, eps=0.02, dtype="c64", want_p1=True)
    e = qs.run_rounds(**kw)
    g1 = qs.run_rounds(graph=True, **kw)
    qs.run_rounds(**dict(kw, seed=74))
    g2 = qs.run_rounds(graph=True, **kw)
    r = qs.run_rounds_async(stream=torch.cuda.Stream(), **kw).wait()
    for g in (g1, g2, r):
        assert np.array_equal(g["records"], e["records"])
        assert np.array_equal(g["final_bits"], e["final_bits"])
        assert np.array_equal(g["p1"], e["p1"])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,mib", [("c128", "4096"), ("c64", "4096"), ("c64", "4")])
def test_flip_matches_plain_passes_batch_d4(monkeypatch, dtype, mib):
    """Lockstep launches of ragged rounds, whole and in groups of 8 registers."""
    print(f"case flip batch d=4 {dtype} {mib}", flush=True)
    monkeypatch.setenv("QECSV_LOCKSTEP_MIB", mib)
    n_sites = qs.template_info(4, "cr")[1]
    R, p, eps = workloads.batch_params(70, n_sites, 75, p=(1e-3, 3e-2), theta=(0.0, 0.1))
    a, b = _both(monkeypatch, lambda: qs.run_batch(4, "cr", R, p, 75, eps_site=eps, dtype=dtype, max_rounds=9))
    assert a["passes_per_round"] == 3


# First and last passes of a trajectory: the first two form the initial state
# instead of reading it (one round: they are two of the five passes; the X
# basis starts from another state), the last one only sums unless the register
# is wanted.
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("rounds", [1, 2])
@pytest.mark.parametrize("xbasis", [False, True])
def test_first_and_last_pass(monkeypatch, rounds, xbasis, dtype):
    n_sites = qs.template_info(5, "cr")[1]
    eps = np.random.default_rng(17).normal(0.0, 0.05, n_sites)
    kw = dict(d=5, gateset="cr", rounds=rounds, n_traj=2, seed=31, p=0.02, eps_site=eps, dtype=dtype, traj0=3,
              want_p1=True, xbasis=xbasis)
    monkeypatch.setenv("QECSV_SPEC", "0")
    want = qs.run_rounds(**kw)
    monkeypatch.delenv("QECSV_SPEC")
    got = qs.run_rounds(**kw)
    kept = qs.run_rounds(want_states=True, **kw)
    # 24 checks a round, some fifty roundings an amplitude each
    tol = 24 * rounds * 50 * (2.0**-53 if dtype == "c128" else 2.0**-24)
    for g in (got, kept):
        assert np.array_equal(g["records"], want["records"])
        assert np.array_equal(g["final_bits"], want["final_bits"])
        assert np.abs(g["p1"] - want["p1"]).max() <= tol


@pytest.mark.gpu
@pytest.mark.parametrize("n_traj", [3, 5])
def test_large_registers_side_by_side(n_traj):
    """complex64 d = 5 trajectories in groups of four and a remainder: the bits
    of each alone."""
    kw = dict(d=5, gateset="cr", rounds=2, seed=41, p=0.01, eps=0.03, dtype="c64", want_p1=True)
    whole = qs.run_rounds(n_traj=n_traj, traj0=6, **kw)
    for t in (0, n_traj - 1):
        one = qs.run_rounds(n_traj=1, traj0=6 + t, **kw)
        assert np.array_equal(one["records"][0], whole["records"][t])
        assert np.array_equal(one["final_bits"][0], whole["final_bits"][t])
        assert np.array_equal(one["p1"][0], whole["p1"][t])
