"""Orders 5-8 on the matrix cores (needs an MI355X): the edges of its
enumeration (subset groups and units that are not full, SNP counts around the
order), of its operand rows (classes around multiples of 96 individuals and of
a step's two halves) and of its rule (one class too large for the shared
accumulator takes the popcount kernel), against the oracle."""
from __future__ import annotations

import math

import numpy as np
import pytest

from parity import check_topk
from synth import random_genotypes

pytestmark = pytest.mark.gpu
CROSS, POPCOUNT = 8, 0  # kernel variants


@pytest.fixture(scope="module")
def cx():
    from paper_2201_02460_amd import epi

    with epi.Context(0) as c:
        yield c


@pytest.mark.parametrize("order,M,N,n_cases,K", [
    (5, 5, 40, 20, 3), (5, 6, 97, 96, 6), (5, 11, 193, 97, 30), (5, 15, 288, 192, 256), (5, 17, 385, 96, 40),
    (6, 6, 30, 10, 2), (6, 8, 96, 95, 28), (6, 11, 291, 98, 20), (6, 13, 576, 288, 50),
    (7, 7, 50, 20, 1), (7, 9, 190, 95, 36), (7, 12, 300, 100, 15),
    (8, 8, 64, 32, 5), (8, 10, 193, 96, 45), (8, 12, 289, 193, 9),
])
def test_cross_kernel_edges(cx, orc, order, M, N, n_cases, K):
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(M, N, seed=31 * order + M, case_fraction=n_cases / N)
    print("case", order, M, N, K, flush=True)
    ds = cx.load(G, y)
    try:
        r = cx.scan(ds, order, K)
        assert r["variant"] == CROSS and len(r["combos"]) == min(K, math.comb(M, order))
        check_topk(orc, G, y, order, K, r["combos"], r["scores"], r["tables"])
        sid = epi.epi_scan_check(cx.ctx, ds, order, K)
        epi.epi_wait(cx.ctx, sid)
        assert epi.epi_scan_digest(cx.ctx, sid) == orc.digest(G, y, order)
        epi.epi_release(cx.ctx, sid)
        ids = epi.epi_scan_batch(cx.ctx, [(ds, order, K), (ds, 2, 3)])  # beside another order, in a graph
        epi.epi_wait(cx.ctx, ids[0])
        c, s, t = epi.epi_results(cx.ctx, ids[0], K, order)
        assert np.array_equal(c, r["combos"]) and np.array_equal(s, r["scores"]) and np.array_equal(t, r["tables"])
        for sid in ids:
            epi.epi_release(cx.ctx, sid)
    finally:
        epi.epi_unload(cx.ctx, ds)


@pytest.mark.parametrize("N,n_cases,variant", [(8190, 4095, CROSS), (8192, 4096, POPCOUNT), (6000, 600, CROSS),
                                               (17000, 300, POPCOUNT)])
def test_cross_kernel_class_size_rule(cx, orc, N, n_cases, variant):
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(7, N, seed=N, case_fraction=n_cases / N)
    ds = cx.load(G, y)
    try:
        r = cx.scan(ds, 5, 10)
        assert r["variant"] == variant
        check_topk(orc, G, y, 5, 10, r["combos"], r["scores"], r["tables"])
    finally:
        epi.epi_unload(cx.ctx, ds)


def test_cross_kernel_without_room(orc):
    """A context whose budget holds the dataset and the scan, but not the cell
    rows of its pairs, still takes the scan (popcount kernel)."""
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(100, 4000, seed=3, case_fraction=0.5)
    G[12:] = 0  # one genotype: few distinct tables, the oracle scans the first SNPs
    with epi.Context(0, 9 << 20) as cx:  # 5 MiB of it a table of the context
        ds = cx.load(G[:12], y)
        few = cx.scan(ds, 5, 5)
        assert few["variant"] == CROSS
        ds2 = cx.load(G[:40], y)
        r = cx.scan(ds2, 5, 5, tables=False)
        assert r["variant"] == POPCOUNT
        check_topk(orc, G[:12], y, 5, 5, few["combos"], few["scores"], few["tables"])
        assert r["scores"][0] >= few["scores"][0]
