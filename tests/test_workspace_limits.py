"""What a bound on the line summaries admits (no GPU): a run that fits in one row band
with whole strips is never cut into more, and a run whose strips fit is never given
column segments that do not."""
import pytest

from test_band_plan import plan
from workloads import Params


def a256(x):
    return (x + 255) // 256 * 256


def whole_strips(n, p, waves, strips):
    """Bytes of a band of `strips` uncut strips: per strip and column, and per strip
    and diagonal, two 2-byte runs; the row leads; the last column tile; the
    statistics; 32 bytes per column tile and the carries where there are bands."""
    H, wp, tiles = 64 * waves, max(p.theiler, 1), (n - 1) // 64 + 1
    total = -(-(n - wp) // H)
    entries = strips * (n - wp) - H * strips * (strips - 1) // 2
    return (a256(4 * (64 + (p.m - 1) * p.tau)) + a256(4 * n) + 4 * a256(2 * entries) + a256(24 * 60)
            + (a256(4 * (64 + 8 * tiles)) if p.m <= 6 else 0) + (2 * a256(4 * n) if strips < total else 0))


@pytest.mark.parametrize("n,limit", [(2_000, 100 << 10), (9_973, 4 << 20), (16_000, 8 << 20)])
def test_one_band_where_whole_strips_fit(n, limit):
    q = plan(Params(m=1, tau=1, eps=0.5, norm=3, theiler=1), n, 0, limit)
    assert q["bands"] == 1 and q["workspace_bytes"] <= limit, q


@pytest.mark.parametrize("waves", [1, 2, 4, 8])
@pytest.mark.parametrize("m,tau,theiler", [(1, 1, 1), (3, 10, 0), (6, 2, 30), (7, 3, 700)])
def test_bound_of_whole_strips(waves, m, tau, theiler):
    p = Params(m=m, tau=tau, eps=0.5, norm=3, theiler=theiler)
    for n in (750, 1_000, 2_003, 4_096, 8_100):      # (fewer than 128 column tiles)
        S = -(-(n - max(theiler, 1)) // (64 * waves))
        for k in {1, 2, S // 2, S - 1, S}:
            if not 1 <= k <= S:
                continue
            limit = whole_strips(n, p, waves, k)
            q = plan(p, n + (m - 1) * tau, waves, limit)
            assert q["workspace_bytes"] <= limit, (n, k, limit, q)
            assert q["bands"] == 1 or k < S, (n, k, q)


@pytest.mark.parametrize("n,waves,segs", [
    (2_000, 0, 16), (12_000, 4, 20), (30_000, 8, 20),    # less than one round of blocks: as many as there may be
    (26_000, 4, 19), (40_000, 8, 18), (56_761, 8, 13),   # one round, not one and a half
    (65_521, 8, 20),                                     # two, and no fewer segments than 64 tiles wide
    (100_000, 8, 24)])
def test_short_segments_do_not_begin_a_round(n, waves, segs):
    q = plan(Params(m=1, tau=1, eps=0.5, norm=3, theiler=1), n, waves, 0)
    # (tiles shared out evenly: the last segment may vanish)
    tiles = (n - 1) // 64 + 1
    assert q["segs"] in (segs, -(-tiles // -(-tiles // segs))), q
