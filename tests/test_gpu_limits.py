"""Runs under a workspace limit (GPU), against the oracle, bit for bit: classified tiles
(128 column tiles and more), short column segments and row bands together, from one
band of whole strips down to bands of one strip, in every shape.  The limit holds, and
what fitted in one band with whole strips takes one."""
import numpy as np
import pytest

from workloads import Params
from test_gpu_tile_ways import check, series
from test_workspace_limits import whole_strips

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [0, 1, 2, 4, 8])
@pytest.mark.parametrize("kind,n,p", [
    ("sine", 2_500, Params(m=2, tau=2, eps=0.8, norm=2, theiler=0)),
    ("uniform", 4_100, Params(m=3, tau=1, eps=0.2, norm=1, theiler=5)),
    ("lorenz", 8_321, Params(m=3, tau=10, eps=0.1, norm=3, theiler=70))])
def test_bounded_runs(cuda, oracle_lib, kind, n, p, waves):
    import torch
    from paper_2402_16853_amd import RQA
    s = series(kind, n + (p.m - 1) * p.tau, 4)
    ref = oracle_lib.histograms(s, p.m, p.tau, p.eps, p.norm, p.theiler)
    H = 64 * (waves or 8)
    S = -(-(n - max(p.theiler, 1)) // H)
    for strips in {S, S // 2, 2, 1}:
        if strips < 1:
            continue
        limit = whole_strips(n, p, H // 64, strips) + (whole_strips(n, p, H // 64, 1) if strips < S else 0)
        print(f"[case] bounded {kind} n={n} waves={waves} limit={limit}", flush=True)
        comp = RQA.from_params(p)
        comp.set_tiling(waves, 0)
        comp.set_workspace_limit(limit)
        check(comp(torch.from_numpy(s).to(cuda)), ref, (kind, n, waves, limit))
        q = comp.last_plan()
        comp.close()
        assert q["workspace_bytes"] <= limit, q
        if waves and strips == S and n < 8_192:
            assert q["bands"] == 1, q


@pytest.mark.parametrize("n,n2,limit", [(700, 8_200, 200 << 10), (3_000, 900, 30 << 10), (9_000, 8_200, 900 << 10)])
def test_bounded_cross(cuda, oracle_lib, n, n2, limit):
    import torch
    from paper_2402_16853_amd import RQA
    p = Params(m=2, tau=3, eps=0.5, norm=2, theiler=40)
    a, b = series("lorenz", n + 3, 1), series("sine", n2 + 3, 2)
    ref = oracle_lib.cross_histograms(a, b, p.m, p.tau, p.eps, p.norm, p.theiler)
    da, db = torch.from_numpy(a).to(cuda), torch.from_numpy(b).to(cuda)
    for waves in (0, 1, 8):
        print(f"[case] bounded cross {n}x{n2} waves={waves}", flush=True)
        comp = RQA.from_params(p)
        comp.set_tiling(waves, 0)
        comp.set_workspace_limit(limit)
        check(comp.cross(da, db), ref, (n, n2, waves))
        comp.close()
