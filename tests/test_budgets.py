"""What a job takes of a server's budget (no GPU): its histograms, its record and its
line summaries, whatever its tiles are pruned with."""
import pytest

from test_workspace_limits import a256, whole_strips
from workloads import Params


@pytest.mark.parametrize("n", [64, 1_000, 8_100])
@pytest.mark.parametrize("m,tau,theiler", [(1, 1, 0), (3, 10, 1), (6, 2, 900), (8, 1, 65)])
def test_footprint_of_short_jobs(n, m, tau, theiler):
    from paper_2402_16853_amd import Server
    theiler = min(theiler, n // 2)
    p = Params(m=m, tau=tau, eps=0.5, norm=3, theiler=theiler)
    strips = -(-(n - max(theiler, 1)) // 256)
    assert Server.footprint(p, n + (m - 1) * tau) == \
        a256(24 * (n + 1)) + 256 + whole_strips(n, p, 4, strips)


def test_footprints_of_long_jobs():
    """(Column segments, strips of four waves below 32,768 vectors and of eight above.)"""
    from paper_2402_16853_amd import Server
    P = Params(m=3, tau=10, eps=0.4, norm=3, theiler=1)
    for n, want in FOOTPRINTS.items():
        assert Server.footprint(P, n) == want, n


FOOTPRINTS = {10_000: 2_882_560, 20_000: 11_084_032, 32_787: 29_308_416, 32_788: 16_728_832, 65_536:
              64_894_208, 200_000: 525_901_056, 1_048_576: 8_623_671_552}
