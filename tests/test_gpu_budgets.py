"""Jobs at the edge of what memory admits them (GPU): a server whose budget is exactly a
job's footprint runs it, and rqa_run_static takes a series of millions of points under
a Theiler window as long.  And Theiler windows about tile and segment edges: what was
written is noted per column tile from the window on."""
import ctypes

import numpy as np
import pytest

from workloads import Params
from test_gpu_tile_ways import check, series

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,theiler", [(700, 2, 1), (8_300, 3, 1), (12_289, 5, 12_289), (30_000, 3, 0),
                                         (90_000, 6, 1), (90_000, 7, 30), (600_000, 3, 599_000)])
def test_job_as_large_as_the_budget(cuda, n, m, theiler):
    import torch
    from paper_2402_16853_amd import RQA, RQAError, Server
    p = Params(m=m, tau=2, eps=0.1 * m, norm=3, theiler=theiler)
    ds = torch.from_numpy(series("uniform", n, n)).to(cuda)
    budget = Server.footprint(p, n)
    comp = RQA.from_params(p)
    ref = comp(ds)
    print(f"[case] budget n={n} m={m} theiler={theiler}", flush=True)
    srv = Server(budget, streams=2)
    for _ in range(2):
        check(srv.wait(srv.submit(p, ds)), (ref.diag, ref.vert, ref.white), (n, m, theiler))
    srv.close()
    if budget > 8192:
        srv = Server(budget - 256, streams=2)
        with pytest.raises(RQAError) as err:
            srv.submit(p, ds)
        assert err.value.code == -8
        srv.close()
    comp.close()


@pytest.mark.parametrize("m,theiler", [(3, 12_000_000), (1, 11_999_000)])
def test_static_run_under_a_long_window(cuda, m, theiler):
    import torch
    from paper_2402_16853_amd import make_params
    from paper_2402_16853_amd._lib import lib
    n = 12_000_000
    hist = torch.full((3 * (n + 1),), -1, dtype=torch.int64, device=cuda)
    flag = torch.full((1,), -1, dtype=torch.int32, device=cuda)
    # nothing recurs: every column is one white line
    ds = torch.arange(n + (m - 1), dtype=torch.float32, device=cuda)
    p = make_params(m, 1, 0.25, 3, theiler=theiler)
    print(f"[case] static n={n} m={m} theiler={theiler}", flush=True)
    rc = lib().rqa_run_static(ctypes.byref(p), ctypes.c_void_p(ds.data_ptr()), ds.numel(),
                              ctypes.c_void_p(hist.data_ptr()), n + 1, ctypes.c_void_p(flag.data_ptr()),
                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    assert flag.item() == 0
    d, v, w = hist.view(3, n + 1)
    assert not d.any() and not v.any()
    assert w[n].item() == n and int(w.sum()) == n


@pytest.mark.parametrize("theiler", [62, 63, 64, 65, 127, 128, 129, 8_000, 8_191, 8_192, 8_193, 8_255, 8_256, 8_320])
@pytest.mark.parametrize("n", [8_256, 8_300])
def test_windows_about_tile_edges(cuda, oracle_lib, n, theiler):
    import torch
    from paper_2402_16853_amd import RQA
    p = Params(m=2, tau=2, eps=0.7, norm=1, theiler=theiler)
    s = series("sine", n + 2, 6)
    ref = oracle_lib.histograms(s, p.m, p.tau, p.eps, p.norm, p.theiler)
    ds = torch.from_numpy(s).to(cuda)
    comp = RQA.from_params(p)
    for waves, limit in ((0, 0), (1, 0), (4, 1 << 20), (2, 1)):
        print(f"[case] window n={n} theiler={theiler} waves={waves} limit={limit}", flush=True)
        comp.set_tiling(waves, 0)
        comp.set_workspace_limit(limit)
        check(comp(ds), ref, (n, theiler, waves, limit))
    comp.close()
