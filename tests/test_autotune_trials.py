"""What the autotuner times, and what it leaves behind when it cannot."""
import numpy as np
import pytest
import torch

import paper_2204_11404_amd as qs

ENV = ("QECSV_ZCHAIN", "QECSV_SNAKE", "QECSV_BATCH_WAVES_PER_CU", "QECSV_LOCKSTEP_MIB", "QECSV_PASS_WGS_PER_CU",
       "QECSV_XPAIR", "QECSV_SPEC")


@pytest.mark.skipif(torch.cuda.is_available(), reason="for a machine without a GPU, where every trial fails")
@pytest.mark.parametrize("d", [3, 4, 5])
def test_failed_trials_leave_the_parameters_untuned(tmp_path, d):
    """An entry left behind would count as tuned, and d = 5 runs that nobody
    tuned choose their chain length themselves."""
    def lines():
        qs.tuning_save(str(tmp_path / "t.txt"))
        return sorted((tmp_path / "t.txt").read_text().splitlines())

    before = lines()
    with pytest.raises(qs.SvError):
        qs.autotune(d, "c64")
    assert lines() == before


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(3, 16384), (4, 4096)])
def test_trials_are_the_batches_that_run(monkeypatch, d, n):
    """The winner's time is that of the two batches it is chosen for, without
    the data ZZ layer and with it, as sv_run_batch runs them.  Within a
    quarter: the same launches, the fastest of two against that of four."""
    for var in ENV:
        monkeypatch.delenv(var, raising=False)
    saved = qs.tuning_get(d, "c64")
    try:
        _, ms = qs.autotune(d, "c64")
        kw = dict(max_rounds=3, eps=0.0125, dtype="c64")
        t = sum(min(qs.run_batch(d, "cr", np.full(n, 3, np.int32), np.full(n, 2e-3), 0x7E57, zeta=z, **kw)["gpu_ms"]
                    for _ in range(4)) for z in (0.0, 0.01))
        print(f"case autotune d={d}: {ms:.3f} ms, batches {t:.3f} ms", flush=True)
        assert 0.75 < ms / t < 1.25
    finally:
        qs.tuning_set(d, "c64", **saved)
