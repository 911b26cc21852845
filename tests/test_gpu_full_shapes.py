"""How full matrices are cut (GPU): as many column segments as it takes to fill the chip,
and no more, and as many waves as their cells ask for; against the oracle."""
import numpy as np
import pytest

from workloads import Params
from test_gpu_tile_ways import check, series

pytestmark = pytest.mark.gpu

P = Params(m=1, tau=1, eps=0.02, norm=3, theiler=3)


@pytest.mark.parametrize("n,n2,rows", [
    (200_000, 1_000, 512),      # 391 strips: two wide segments, and 1,024 items ask for three
    (2_048, 66_000, 512),       # many cells behind few rows: eight waves
    (2_047, 66_000, 256),       # four
    (3_000, 1_300, 256)])       # short chains: a twentieth each
def test_cut_of_a_cross_matrix(cuda, oracle_lib, n, n2, rows):
    import torch
    from paper_2402_16853_amd import RQA
    a, b = series("uniform", n, 1), series("uniform", n2, 2)
    print(f"[case] cut of {n}x{n2}", flush=True)
    comp = RQA.from_params(P)
    res = comp.cross(torch.from_numpy(a).to(cuda), torch.from_numpy(b).to(cuda))
    plan = comp.last_plan()
    comp.close()
    assert plan["strip_rows"] == rows, plan
    strips, tiles = -(-n // rows), -(-n2 // 64)
    segs = max(1, tiles // 8, min(-(-1024 // strips), tiles // max(1, min(8, tiles // 20))))
    width = -(-tiles // segs)
    assert plan["segs"] == -(-tiles // width), plan
    check(res, oracle_lib.cross_histograms(a, b, P.m, P.tau, P.eps, P.norm, P.theiler), (n, n2))


@pytest.mark.parametrize("n,rows", [(24_575, 256), (24_576, 512)])
def test_shape_of_a_given_matrix(cuda, oracle_lib, n, rows):
    import torch
    from paper_2402_16853_amd import RQA
    nb = 700
    rng = np.random.default_rng(n)
    bits = rng.integers(0, 1 << 64, size=(n, 11), dtype=np.uint64)
    print(f"[case] given matrix of {n} rows", flush=True)
    comp = RQA.from_params(P)
    res = comp.matrix(torch.from_numpy(bits.view(np.int64)).to(cuda), nb)
    plan = comp.last_plan()
    comp.close()
    assert plan["strip_rows"] == rows, plan
    check(res, oracle_lib.matrix_histograms(bits, n, nb, P.theiler), n)


@pytest.mark.parametrize("waves", [1, 4, 8])
@pytest.mark.parametrize("eps", [2e-5, 2e-4, 1e-3])
def test_tiles_of_few_cells(cuda, oracle_lib, eps, waves):
    """Noise that leaves a tile no cell, a few rows with one, or most rows: one series and
    a cross pair."""
    import torch
    from paper_2402_16853_amd import RQA
    p = Params(m=1, tau=1, eps=eps, norm=3, theiler=0)
    a, b = series("uniform", 1_500, 1), series("uniform", 1_111, 2)
    da, db = torch.from_numpy(a).to(cuda), torch.from_numpy(b).to(cuda)
    print(f"[case] few cells eps={eps} waves={waves}", flush=True)
    comp = RQA.from_params(p)
    comp.set_tiling(waves, 0)
    check(comp(da), oracle_lib.histograms(a, 1, 1, p.eps, 3, 0), (eps, waves))
    check(comp.cross(da, db), oracle_lib.cross_histograms(a, b, 1, 1, p.eps, 3, 0), (eps, waves, "cross"))
    comp.close()
