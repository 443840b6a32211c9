"""sv_run_batch at d = 3 without the data ZZ layer: the register in one wave's
registers, the checks of a round in two chains (k_batch_flip), against the
circuit-by-circuit kernel (QECSV_BATCH_SPLIT=1), which the oracle checks.
Records and final bits must agree bit for bit; p up to 0.1 draws Paulis in
every round, so both frames and rebuilt Kraus pairs take part."""
import numpy as np
import pytest

import paper_2204_11404_amd as qs
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("gateset", ["cr", "textbook"])
@pytest.mark.parametrize("n,p,shared", [(1, (0.05, 0.1), False), (777, (0.0, 0.1), False), (2500, (5e-4, 5e-3), False),
                                        (300, (0.02, 0.05), True)])
def test_batch_flip_matches_circuits(monkeypatch, dtype, gateset, n, p, shared):
    """One trajectory; ragged rounds over fewer and more trajectories than the
    grid holds at once (one resident wave per compute unit); angles of their
    own and common ones."""
    print(f"case batch flip {gateset} {dtype} n={n} p={p} shared={shared}", flush=True)
    monkeypatch.setenv("QECSV_BATCH_WAVES_PER_CU", "1")
    n_sites = qs.template_info(3, gateset)[1]
    R, pp, eps = workloads.batch_params(n, n_sites, 91, p=p, theta=(0.0, 0.3))
    kw = dict(max_rounds=9, dtype=dtype, eps=0.07) if shared else dict(max_rounds=9, dtype=dtype, eps_site=eps)
    out = []
    for split in (None, "1"):
        monkeypatch.delenv("QECSV_BATCH_SPLIT", raising=False)
        if split:
            monkeypatch.setenv("QECSV_BATCH_SPLIT", split)
        out.append(qs.run_batch(3, gateset, R, pp, 91, **kw))
    assert np.array_equal(out[0]["records"], out[1]["records"])
    assert np.array_equal(out[0]["final_bits"], out[1]["final_bits"])
