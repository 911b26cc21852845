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


@pytest.mark.parametrize("n,n2", [(16_500, 8_200), (8_200, 16_500), (270_000, 2_100)])
def test_classified_tall_cross(cuda, oracle_lib, n, n2):
    """Boxes of rows and columns that are not the same, over several strips and column
    segments; 33 column tiles are enough behind 131,072 tiles in all."""
    import torch
    from paper_2402_16853_amd import RQA
    for kind, p in (("sine", Params(m=2, tau=3, eps=0.8, norm=2, theiler=0)),
                    ("lorenz", Params(m=3, tau=10, eps=0.1, norm=3, theiler=100))):
        lag = (p.m - 1) * p.tau
        a, b = series(kind, n + lag, 1), series(kind, n2 + lag, 2)
        print(f"[case] tall cross {n}x{n2} {kind}", flush=True)
        comp = RQA.from_params(p)
        res = comp.cross(torch.from_numpy(a).to(cuda), torch.from_numpy(b).to(cuda))
        comp.close()
        check(res, oracle_lib.cross_histograms(a, b, p.m, p.tau, p.eps, p.norm, p.theiler), (n, n2, kind))


@pytest.mark.parametrize("kind,p", [("sine", Params(m=3, tau=2, eps=0.3, norm=2, theiler=0)),
                                    ("lorenz", Params(m=2, tau=5, eps=0.1, norm=3, theiler=70)),
                                    ("uniform", Params(m=5, tau=1, eps=0.5, norm=1, theiler=1))])
def test_classified_windows(cuda, oracle_lib, kind, p):
    """Windows about the 32 column tiles from which those of a batch are classified, and
    the same lengths as served jobs."""
    import torch
    from paper_2402_16853_amd import RQA, Server
    lag = (p.m - 1) * p.tau
    ln = np.array([31 * 64, 31 * 64 + 1, 32 * 64, 40 * 64 + 5, 700, 5_000], dtype=np.int64) + lag
    off = np.arange(len(ln), dtype=np.int64) * 100
    s = series(kind, int(5_600 + lag), 4)
    ds = torch.from_numpy(s).to(cuda)
    ref = [oracle_lib.histograms(s[o:o + k], p.m, p.tau, p.eps, p.norm, p.theiler) for o, k in zip(off, ln)]
    comp = RQA.from_params(p)
    for waves in (0, 1, 2, 8):
        print(f"[case] classified windows {kind} waves={waves}", flush=True)
        comp.set_tiling(waves, 0)
        comp.run_batch(ds, off, ln)
        for w in range(len(ln)):
            check(comp.result_batch(w), ref[w], (kind, waves, w))
    comp.close()
    srv = Server(64 << 20, streams=2)
    tickets = [srv.submit(p, ds[o:o + k].clone()) for o, k in zip(off, ln)]
    for w, t in enumerate(tickets):
        check(srv.wait(t), ref[w], (kind, "served", w))
    srv.close()
