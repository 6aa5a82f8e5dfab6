"""The popcount kernel of orders 5-8 (needs an MI355X): the fallback of scans
that the matrix-core kernel does not take.  Pinned with EPI_BLOCK_ALL_CELLS it
scores every combination once with the oracle's table, at small sizes and at
the named workloads, and gives the matrix-core kernel's results; classes too
large for the matrix-core kernel reach it unpinned."""
from __future__ import annotations

import json
import math
import os

import numpy as np
import pytest

from parity import check_topk
from synth import make_workload, random_genotypes

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")
CROSS, POPCOUNT = 8, 0  # kernel variants


@pytest.fixture(scope="module")
def cx():
    from paper_2201_02460_amd import epi

    with epi.Context(0) as c:
        yield c


def checked(cx, ds, order, K):
    """(digest, results, variant) of a checking scan."""
    from paper_2201_02460_amd import epi

    sid = epi.epi_scan_check(cx.ctx, ds, order, K)
    try:
        epi.epi_wait(cx.ctx, sid)
        return (epi.epi_scan_digest(cx.ctx, sid), epi.epi_results(cx.ctx, sid, K, order),
                epi.epi_scan_info(cx.ctx, sid)["variant"])
    finally:
        epi.epi_release(cx.ctx, sid)


def pinned_equals_default(cx, ds, order, K):
    from paper_2201_02460_amd import epi

    dig, res, variant = checked(cx, ds, order, K)
    assert variant == CROSS
    epi.epi_set_prefix_block(cx.ctx, ds, order, epi.EPI_BLOCK_ALL_CELLS)
    try:
        pdig, pres, variant = checked(cx, ds, order, K)
        assert variant == POPCOUNT
        plain = cx.scan(ds, order, K)
        assert plain["variant"] == POPCOUNT
    finally:
        epi.epi_set_prefix_block(cx.ctx, ds, order, 0)
    assert pdig == dig
    for a, b, c in zip(res, pres, (plain["combos"], plain["scores"], plain["tables"])):
        assert np.array_equal(a, b) and np.array_equal(a, c)
    return dig


@pytest.mark.parametrize("order,M,N,n_cases", [(5, 22, 200, 60), (5, 9, 97, 31), (6, 14, 130, 40), (7, 12, 96, 48),
                                               (8, 13, 260, 100)])
def test_pinned_popcount_digest(cx, orc, order, M, N, n_cases):
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(M, N, seed=300 + M + order, case_fraction=n_cases / N)
    print("case", order, M, N, flush=True)
    ds = cx.load(G, y)
    try:
        assert pinned_equals_default(cx, ds, order, 12) == orc.digest(G, y, order)
    finally:
        epi.epi_unload(cx.ctx, ds)


@pytest.mark.parametrize("name", ["order5_M60_N2000", "order8_M23_N2048"])
def test_pinned_popcount_full_size(cx, name):
    from paper_2201_02460_amd import epi

    with open(os.path.join(GOLDEN, "digest_" + name + ".json")) as f:
        gold = json.load(f)
    G, y, spec, _ = make_workload(name)
    ds = cx.load(G, y)
    try:
        dig = pinned_equals_default(cx, ds, spec["order"], spec["top_k"])
        assert dig == (gold["n_combinations"], gold["digest"])
    finally:
        epi.epi_unload(cx.ctx, ds)


@pytest.mark.parametrize("order,M", [(5, 8), (6, 8), (7, 9), (8, 10)])
def test_popcount_of_large_classes(cx, orc, order, M):
    """4096 individuals in one class: the unpinned scan's kernel."""
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(M, 8192, seed=order, case_fraction=0.5)
    print("case", order, M, flush=True)
    ds = cx.load(G, y)
    try:
        dig, res, variant = checked(cx, ds, order, 20)
        assert variant == POPCOUNT and dig == orc.digest(G, y, order)
        assert len(res[0]) == min(20, math.comb(M, order))
        check_topk(orc, G, y, order, 20, *res)
    finally:
        epi.epi_unload(cx.ctx, ds)


def test_popcount_without_room_finds_the_same(orc):
    """A scan whose cell rows do not fit the context's budget returns the same
    best combinations: SNPs of one genotype add nothing to a combination, so
    those of the panel without them."""
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(40, 4000, seed=3, case_fraction=0.5)
    G[12:] = 0
    with epi.Context(0, 9 << 20) as cx:  # 5 MiB of it a table of the context
        few = cx.scan(cx.load(G[:12], y), 5, 5)
        r = cx.scan(cx.load(G, y), 5, 5)
    assert few["variant"] == CROSS and r["variant"] == POPCOUNT
    for k in ("combos", "scores", "tables"):
        assert np.array_equal(few[k], r[k])
    check_topk(orc, G[:12], y, 5, 5, r["combos"], r["scores"], r["tables"])
