"""The largest launches that the no-allocation batch takes: its 64 MiB count the
tables, parameters and results of a job, not how a kernel lays them out."""
import numpy as np
import pytest

import paper_2204_11404_amd as qs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,gateset,dtype,per_site,max_rounds,most", [
    (3, "cr", "c64", True, 9, 119561), (3, "cr", "c128", False, 9, 593511), (3, "textbook", "c64", True, 1, 378952),
    (2, "cr", "c64", True, 4, 322496), (3, "textbook", "c128", False, 30, 238675)])
def test_largest_launch(d, gateset, dtype, per_site, max_rounds, most):
    print(f"case no-alloc limit {d} {gateset} {dtype} {max_rounds}", flush=True)
    sites = qs.template_info(d, gateset)[1]

    def run(n, no_alloc=True):
        kw = dict(eps_site=np.full((n, sites), 0.02)) if per_site else dict(eps=0.02)
        return qs.run_batch(d, gateset, np.ones(n, np.int32), np.full(n, 0.01), 1, dtype=dtype, max_rounds=max_rounds,
                            no_alloc=no_alloc, **kw)

    a, b = run(most), run(most, no_alloc=False)
    assert np.array_equal(a["records"], b["records"])
    assert np.array_equal(a["final_bits"], b["final_bits"])
    with pytest.raises(qs.SvError) as e:
        run(most + 1)
    assert e.value.status == qs.SV_ENOMEM
