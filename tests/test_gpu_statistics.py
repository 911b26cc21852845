"""The histogram statistics at the edges of their blocks (GPU): 2,048 lengths are
one block's work, done by one kernel; a longer histogram takes a second kernel
whose last block adds the partial sums up.  The white histogram of a series with
an isolated first vector fills the last length.  Histograms against the oracle
(exact), measures within 1e-12 (a sum of at most 2,049 terms rounds far below
that); a non-finite value is reported on both sides of the edge."""
import numpy as np
import pytest

from workloads import Params
from test_gpu_parity import assert_same, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 255, 2046, 2047, 2048, 2049, 4097])
def test_statistics_block_edges(cuda, oracle_lib, n):
    rng = np.random.default_rng(n)
    s = rng.random(n + 1).astype(np.float32)
    s[0] = 50.0                      # recurs with nothing: a white line over the column
    p = Params(m=2, tau=1, eps=0.2, norm=3, lmin=2, vmin=3, wmin=n, theiler=1)
    print(f"[case] statistics n={n}", flush=True)
    res = run_gpu(s, p, cuda)
    ref_hist, ref_meas = oracle_lib.rqa(s, p)
    assert_same(res, ref_hist, ref_meas, f"n={n}")


@pytest.mark.parametrize("n", [2047, 2049])
def test_non_finite_is_reported(cuda, n):
    from paper_2402_16853_amd._lib import RQAError
    s = np.linspace(0, 1, n).astype(np.float32)
    s[n - 1] = np.inf
    print(f"[case] non-finite n={n}", flush=True)
    with pytest.raises(RQAError) as err:
        run_gpu(s, Params(m=1, tau=1, eps=0.1, norm=1), cuda)
    assert err.value.code == -5
