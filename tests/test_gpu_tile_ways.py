"""The tile kernel's ways at their edges (GPU), against the oracle, bit for bit:

* short runs cut into up to 20 column segments (1 tile wide at the smallest; 20
  and 21 column tiles; one more and one less than a tile), in every shape;
* tiles classified from boxes: jobs of 127 and 128 column tiles (128 is the
  first to take boxes), series with fully recurrent tiles (sine), mostly empty
  ones (Lorenz) and none to decide (noise), every norm, ragged ends, Theiler
  windows that cut the classes' groups, m above and below the three
  coordinates a box holds;
* batches of few windows, whose chains are cut as well."""
import numpy as np
import pytest

from workloads import Params, lorenz_x_series

pytestmark = pytest.mark.gpu


def series(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "sine":
        return np.sin(np.linspace(0.0, 0.01 * n, n) + rng.uniform(0, 6)).astype(np.float32)
    if kind == "lorenz":
        s = lorenz_x_series(n, seed).astype(np.float64)
        return (s / s.std()).astype(np.float32)
    if kind == "constant":
        return np.full(n, 0.25, dtype=np.float32)
    return rng.random(n).astype(np.float32)


def check(res, ref, tag):
    for name, a, b in zip(("diag", "vert", "white"), (res.diag, res.vert, res.white), ref):
        assert np.array_equal(a, b), f"{tag}: {name} differs at {np.nonzero(a != b)[0][:8]}"


@pytest.mark.parametrize("n", [63, 64, 65, 129, 1280, 1281, 1345, 2600])
@pytest.mark.parametrize("waves", [1, 2, 4, 8])
def test_short_runs_in_segments(cuda, oracle_lib, n, waves):
    import torch
    from paper_2402_16853_amd import RQA
    for kind, p in (("uniform", Params(m=2, tau=1, eps=0.25, norm=2, theiler=1)),
                    ("sine", Params(m=2, tau=2, eps=0.6, norm=1, theiler=0)),
                    ("constant", Params(m=1, tau=1, eps=0.1, norm=3, theiler=7))):
        s = series(kind, n + (p.m - 1) * p.tau, n + waves)
        print(f"[case] segments n={n} waves={waves} {kind}", flush=True)
        comp = RQA.from_params(p)
        comp.set_tiling(waves, 0)
        res = comp(torch.from_numpy(s).to(cuda))
        assert comp.last_plan()["segs"] > 1 or n <= 64 * 2
        comp.close()
        check(res, oracle_lib.histograms(s, p.m, p.tau, p.eps, p.norm, p.theiler), (n, waves, kind))


@pytest.mark.parametrize("n", [127 * 64, 127 * 64 + 1, 8500])
@pytest.mark.parametrize("kind,m,tau,eps,norm,theiler", [
    ("sine", 1, 1, 0.5, 3, 1), ("sine", 2, 2, 1.0, 2, 0), ("sine", 3, 5, 1.2, 1, 300),
    ("lorenz", 3, 10, 0.05, 3, 30), ("lorenz", 3, 7, 0.2, 2, 1), ("lorenz", 4, 5, 0.4, 1, 65),
    ("lorenz", 5, 3, 0.3, 2, 1), ("uniform", 3, 1, 0.2, 3, 1), ("uniform", 6, 2, 0.5, 1, 0),
    ("constant", 2, 1, 0.5, 2, 1)])
def test_classified_tiles(cuda, oracle_lib, n, kind, m, tau, eps, norm, theiler):
    import torch
    from paper_2402_16853_amd import RQA
    p = Params(m=m, tau=tau, eps=eps, norm=norm, theiler=theiler)
    s = series(kind, n + (m - 1) * tau, 5)
    print(f"[case] classes n={n} {kind} m={m} norm={norm} theiler={theiler}", flush=True)
    ref = oracle_lib.histograms(s, m, tau, p.eps, norm, theiler)
    comp = RQA.from_params(p)
    for waves in (0, 8):
        comp.set_tiling(waves, 0)
        check(comp(torch.from_numpy(s).to(cuda)), ref, (n, kind, m, norm, theiler, waves))
    comp.close()


@pytest.mark.parametrize("n,n2", [(700, 8200), (8200, 700)])
def test_classified_cross(cuda, oracle_lib, n, n2):
    import torch
    from paper_2402_16853_amd import RQA
    for kind, p in (("sine", Params(m=2, tau=3, eps=0.8, norm=2, theiler=0)),
                    ("lorenz", Params(m=3, tau=10, eps=0.1, norm=3, theiler=100))):
        lag = (p.m - 1) * p.tau
        a, b = series(kind, n + lag, 1), series(kind, n2 + lag, 2)
        print(f"[case] classes cross {n}x{n2} {kind}", flush=True)
        comp = RQA.from_params(p)
        res = comp.cross(torch.from_numpy(a).to(cuda), torch.from_numpy(b).to(cuda))
        comp.close()
        check(res, oracle_lib.cross_histograms(a, b, p.m, p.tau, p.eps, p.norm, p.theiler), (n, n2, kind))


@pytest.mark.parametrize("count", [2, 9])
def test_batches_of_few_windows(cuda, oracle_lib, count):
    import torch
    from paper_2402_16853_amd import RQA
    rng = np.random.default_rng(count)
    s = series("uniform", 12_000, 3)
    ln = rng.integers(130, 6000, size=count).astype(np.int64)
    ln[0] = 5                                   # fewer vectors than a tile
    off = np.array([rng.integers(0, len(s) - k + 1) for k in ln], dtype=np.int64)
    p = Params(m=2, tau=2, eps=0.1, norm=3, theiler=1)
    comp = RQA.from_params(p)
    ds = torch.from_numpy(s).to(cuda)
    for run in range(4):                        # trials, then a replayed graph
        print(f"[case] few windows {count} run {run}", flush=True)
        comp.run_batch(ds, off, ln)
        for w in range(count):
            ref = oracle_lib.histograms(s[off[w]:off[w] + ln[w]], p.m, p.tau, p.eps, p.norm, p.theiler)
            check(comp.result_batch(w), ref, (count, run, w))
    comp.close()


@pytest.mark.parametrize("rows", [0, 1, 2, 4, 5])
@pytest.mark.parametrize("waves", [1, 8])
def test_tiles_of_few_rows(cuda, oracle_lib, rows, waves):
    """Tiles with a handful of non-zero rows (4 is the last that is gathered row by
    row, 5 the first that is transposed), whole rows and scattered cells among them,
    at both ends and on both sides of row 32."""
    import torch
    from paper_2402_16853_amd import RQA
    n, nb = 600, 700
    rng = np.random.default_rng(10 * rows + waves)
    dense = np.zeros((n, 11 * 64), dtype=np.uint8)
    for r0 in range(0, n, 64):
        near = [r for r in (0, 31, 32, 63) if r0 + r < n]
        pick = near[:rows] + list(rng.choice([r for r in range(1, min(31, n - r0))], max(0, rows - len(near)), False))
        for r in pick:
            dense[r0 + r, :nb] = rng.random(nb) < (1.0 if rng.random() < 0.3 else 0.2)
    print(f"[case] few rows={rows} waves={waves}", flush=True)
    bits = np.packbits(dense, axis=1, bitorder="little").view(np.int64)
    comp = RQA.from_params(Params(m=1, tau=1, eps=0.0, norm=3, theiler=0))
    comp.set_tiling(waves, 0)
    res = comp.matrix(torch.from_numpy(bits).to(cuda), nb)
    comp.close()
    check(res, oracle_lib.matrix_histograms(bits.view(np.uint64), n, nb, 0), (rows, waves))
