"""The autotuner's times of small scans are those of the scans themselves
(needs an MI355X): a scan of a pinned kernel takes, per combination, about
what the tuner reported for it, and the chosen kernel is not slower than the
untuned one.  Both lines are a factor of two, several times the spread of a
100 us kernel and half of what a missing pilot pass makes."""
from __future__ import annotations

import math

import pytest

from synth import random_genotypes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cx():
    from paper_2201_02460_amd import epi

    with epi.Context(0) as c:
        yield c


def main_ns(cx, ds, order, M, K=16, n=9):
    """Median nanoseconds a combination of the scan's main kernel (and pilot)."""
    from paper_2201_02460_amd import epi

    t = []
    for _ in range(n):
        sid = epi.epi_scan(cx.ctx, ds, order, K)
        epi.epi_wait(cx.ctx, sid)
        t.append(epi.epi_scan_timing(cx.ctx, sid)[2])
        epi.epi_release(cx.ctx, sid)
    return sorted(t)[n // 2] * 1e6 / math.comb(M, order)


@pytest.mark.parametrize("order,M,N", [(2, 300, 1500), (3, 151, 1237), (3, 90, 3000), (3, 740, 1955), (4, 60, 900),
                                       (5, 25, 800), (7, 16, 600)])
def test_small_scan_tuned_as_it_runs(cx, order, M, N):
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(M, N, seed=M + N, case_fraction=0.4)
    ds = cx.load(G, y)
    try:
        before = main_ns(cx, ds, order, M)
        choice = epi.epi_autotune(cx.ctx, ds, order)
        after = main_ns(cx, ds, order, M)
        rep = epi.epi_autotune_report(cx.ctx, ds, order)
        print("case", order, M, N, "choice", choice, "report", rep, "before", before, "after", after, flush=True)
        assert after <= 2 * before
        for block, ns in rep:
            epi.epi_set_prefix_block(cx.ctx, ds, order, 0 if order >= 5 and block == epi.EPI_BLOCK_ALL_CELLS else block)
            assert 0.5 < main_ns(cx, ds, order, M) / ns < 2, block
    finally:
        epi.epi_set_prefix_block(cx.ctx, ds, order, 0)
        epi.epi_unload(cx.ctx, ds)
