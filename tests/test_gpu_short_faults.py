"""The give-up path of the bounded waits with few white bins (GPU): jobs of fewer than
960 lengths, whose LDS bins for white lines are fewer than the lengths that arbitrary
states can name.  Every wait is made to give up from the host, as in
test_gpu_faults.py; every kernel runs to its end, the job reports RQA_EDEVICE, and the
next run is exact."""
import numpy as np
import pytest

from workloads import Params
from test_gpu_tile_ways import check, series

pytestmark = pytest.mark.gpu

P = Params(m=2, tau=1, eps=0.2, norm=3, theiler=1)


@pytest.mark.parametrize("n", [62, 130, 500, 958])
@pytest.mark.parametrize("waves", [2, 8])
def test_short_run_gives_up(cuda, oracle_lib, monkeypatch, n, waves):
    import torch
    from paper_2402_16853_amd import RQA
    from paper_2402_16853_amd._lib import RQAError
    s = series("uniform", n + 1, n)
    ds = torch.from_numpy(s).to(cuda)
    comp = RQA.from_params(P)
    comp.set_tiling(waves, 0)
    print(f"[case] short give-up n={n} waves={waves}", flush=True)
    monkeypatch.setenv("RQA_DEBUG_WAIT_GIVEUP", "1")
    with pytest.raises(RQAError) as err:
        comp(ds)
    assert err.value.code == -4
    monkeypatch.delenv("RQA_DEBUG_WAIT_GIVEUP")
    check(comp(ds), oracle_lib.histograms(s, P.m, P.tau, P.eps, P.norm, P.theiler), (n, waves))
    comp.close()


def test_short_windows_give_up(cuda, oracle_lib, monkeypatch):
    import torch
    from paper_2402_16853_amd import RQA
    s = series("uniform", 3_000, 2)
    off = np.arange(40, dtype=np.int64) * 50
    ln = 60 + 20 * np.arange(40, dtype=np.int64)
    ds = torch.from_numpy(s).to(cuda)
    comp = RQA.from_params(P)
    comp.set_tiling(4, 0)
    print("[case] short give-up, windows", flush=True)
    monkeypatch.setenv("RQA_DEBUG_WAIT_GIVEUP", "1")
    comp.run_batch(ds, off, ln)
    _, status = comp.results_batch()
    assert (status == -4).all(), status
    monkeypatch.delenv("RQA_DEBUG_WAIT_GIVEUP")
    comp.run_batch(ds, off, ln)
    for w in range(len(off)):
        check(comp.result_batch(w), oracle_lib.histograms(s[off[w]:off[w] + ln[w]], P.m, P.tau, P.eps, P.norm,
                                                          P.theiler), w)
    comp.close()
