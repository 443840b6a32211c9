"""Batches against a second implementation, where the default one has moved to
kernels that single runs share."""
import numpy as np
import pytest

import oracle
import paper_2204_11404_amd as qs
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("gateset", ["cr", "textbook"])
@pytest.mark.parametrize("d,zeta", [(2, 0.0), (3, 0.0), (3, 0.01)])
def test_batch_matches_register_passes(monkeypatch, d, zeta, gateset, dtype):
    """sv_run_rounds by register passes (a run of d <= 3 takes the batch's
    kernels otherwise)."""
    print(f"case batch and passes d={d} {gateset} {dtype} zeta={zeta}", flush=True)
    n = 64
    eps = workloads.eps_sites(qs.template_info(d, gateset)[1], (0, 0.05), 4)
    a = qs.run_batch(d, gateset, np.full(n, 4, np.int32), np.full(n, 0.02), 4, eps_site=np.tile(eps, (n, 1)),
                     zeta=zeta, traj0=100, dtype=dtype)
    monkeypatch.setenv("QECSV_SPEC", "0")
    b = qs.run_rounds(d, gateset, 4, n, 4, 0.02, eps_site=eps, zeta=zeta, traj0=100, dtype=dtype)
    assert np.array_equal(a["records"], b["records"])
    assert np.array_equal(a["final_bits"], b["final_bits"])


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_predicted_passes_in_several_groups(monkeypatch, dtype):
    """d = 4 in lockstep with predicted outcomes, two registers a slot and one
    or two slots a group: partial sums, tickets and control records are used
    again from group to group."""
    print(f"case predicted groups {dtype}", flush=True)
    monkeypatch.setenv("QECSV_SPEC", "1")
    monkeypatch.setenv("QECSV_LOCKSTEP_MIB", "2")
    n = 16
    R, p, eps = workloads.batch_params(n, qs.template_info(4, "cr")[1], 81, p=(5e-4, 2e-2))
    g = qs.run_batch(4, "cr", R, p, 81, eps_site=eps, dtype=dtype, max_rounds=9)
    assert g["redo_passes"] > 0
    for i in range(n):
        o = oracle.run_trajectory(4, oracle.GATESET_CR, int(R[i]), 81, i, p[i], eps_site=eps[i])
        assert np.array_equal(g["records"][i, :R[i]], o["records"]), f"trajectory {i}"
        assert not g["records"][i, R[i]:].any()
        assert np.array_equal(g["final_bits"][i], o["final_bits"]), f"trajectory {i}"
