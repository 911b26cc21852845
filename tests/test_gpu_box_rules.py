"""Which jobs are classified from boxes, and by what samples (GPU): series that are smooth
in one part and noise in another, so that the samples and the tiles disagree; as few
vectors as a sample needs; values whose distances overflow.  Against the oracle, bit
for bit."""
import numpy as np
import pytest

from workloads import Params
from test_gpu_tile_ways import check, series

pytestmark = pytest.mark.gpu


def mixed(n, seed, part):
    """Smooth but for `part` of it, which is noise."""
    s = series("sine", n, seed)
    k = int(n * part)
    s[n - k:] = series("uniform", k, seed + 1)
    return s


@pytest.mark.parametrize("part", [0.0, 0.2, 0.9, 1.0])
@pytest.mark.parametrize("m,tau,eps,norm,theiler", [(1, 1, 0.05, 3, 1), (3, 4, 0.3, 2, 0), (5, 2, 0.6, 1, 200)])
def test_partly_smooth_series(cuda, oracle_lib, part, m, tau, eps, norm, theiler):
    import torch
    from paper_2402_16853_amd import RQA
    n = 8_192 + 77
    p = Params(m=m, tau=tau, eps=eps, norm=norm, theiler=theiler)
    s = mixed(n + (m - 1) * tau, 3, part)
    print(f"[case] partly smooth part={part} m={m} norm={norm}", flush=True)
    comp = RQA.from_params(p)
    res = comp(torch.from_numpy(s).to(cuda))
    comp.close()
    check(res, oracle_lib.histograms(s, m, tau, p.eps, norm, theiler), (part, m, norm))


@pytest.mark.parametrize("norm,eps", [(1, 1e30), (2, 1e18), (2, 3e19), (3, 2e38)])
def test_distances_that_overflow(cuda, oracle_lib, norm, eps):
    """fl(eps * eps) and distances beyond the largest float: infinite lower and upper
    bounds, and an infinite threshold."""
    import torch
    from paper_2402_16853_amd import RQA
    p = Params(m=2, tau=1, eps=eps, norm=norm, theiler=1)
    s = series("sine", 8_300, 9)
    s[2_000:4_000] *= np.float32(3e38)
    s[6_000:] *= np.float32(1e19)
    print(f"[case] overflow norm={norm} eps={eps}", flush=True)
    comp = RQA.from_params(p)
    res = comp(torch.from_numpy(s).to(cuda))
    comp.close()
    check(res, oracle_lib.histograms(s, p.m, p.tau, p.eps, norm, 1), (norm, eps))
