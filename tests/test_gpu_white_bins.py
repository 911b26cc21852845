"""White lines about the lengths that a workgroup counts in its LDS (GPU): 6,015 at most,
and 4,991 in launches of up to four waves that fill the chip; longer ones are counted
in memory.  Sparse noise has them at every length.  Against the oracle, bit for bit."""
import numpy as np
import pytest

from workloads import Params
from test_gpu_tile_ways import check, series

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [1, 2, 4, 8])
def test_white_lengths_about_the_bins(cuda, oracle_lib, waves):
    import torch
    from paper_2402_16853_amd import RQA
    p = Params(m=1, tau=1, eps=1e-4, norm=3, theiler=1)
    s = series("uniform", 9_000, 5)
    ds = torch.from_numpy(s).to(cuda)
    # 120 windows of 32 strips of four waves: about 2,000 blocks of a whole strip
    ln = np.full(120, 8_000, dtype=np.int64)
    off = np.linspace(0, 1_000, 120).astype(np.int64)
    ln[7], ln[8], ln[9] = 4_991, 4_993, 6_016
    print(f"[case] white lengths of windows, waves={waves}", flush=True)
    comp = RQA.from_params(p)
    comp.set_tiling(waves, 0)
    comp.run_batch(ds, off, ln)
    for w in (0, 7, 8, 9, 119):
        o, k = off[w], ln[w]
        check(comp.result_batch(w), oracle_lib.histograms(s[o:o + k], 1, 1, p.eps, 3, 1), (waves, w))
    # one series of few blocks, and a cross matrix of many
    print(f"[case] white lengths of one series and a cross pair, waves={waves}", flush=True)
    check(comp(ds), oracle_lib.histograms(s, 1, 1, p.eps, 3, 1), (waves, "series"))
    a, b = s[:7_000], series("uniform", 20_000, 6)
    check(comp.cross(torch.from_numpy(a).to(cuda), torch.from_numpy(b).to(cuda)),
          oracle_lib.cross_histograms(a, b, 1, 1, p.eps, 3, 1), (waves, "cross"))
    comp.close()
