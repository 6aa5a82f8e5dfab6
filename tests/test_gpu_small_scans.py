"""Scans of few work items (needs an MI355X): the pilot pass covers up to the
whole scan there, counts per lane when there are fewer items than 4 K, and
must leave the best K as they are -- K from one to past C(M, k), item counts
that are no multiple of a workgroup's four, and both sides of the order-2
rule on the number of individuals."""
from __future__ import annotations

import math

import numpy as np
import pytest

from parity import check_topk
from synth import random_genotypes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cx():
    from paper_2201_02460_amd import epi

    with epi.Context(0) as c:
        yield c


@pytest.mark.parametrize("order,M,N,n_cases,K", [
    (2, 2, 64, 30, 1), (2, 5, 130, 64, 256), (2, 66, 6000, 2100, 40), (2, 66, 6001, 2100, 40), (2, 129, 500, 77, 3),
    (3, 3, 70, 20, 4), (3, 17, 200, 90, 256), (3, 33, 129, 1, 5), (3, 49, 700, 333, 100), (3, 97, 300, 120, 1),
    (4, 4, 80, 40, 2), (4, 12, 300, 100, 256), (4, 29, 222, 111, 60),
])
def test_small_scan_matches_oracle(cx, orc, order, M, N, n_cases, K):
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(M, N, seed=7 * M + order, case_fraction=n_cases / N)
    print("case", order, M, N, K, flush=True)
    ds = cx.load(G, y)
    try:
        r = cx.scan(ds, order, K)
        assert len(r["combos"]) == min(K, math.comb(M, order))
        check_topk(orc, G, y, order, K, r["combos"], r["scores"], r["tables"])
        ids = epi.epi_scan_batch(cx.ctx, [(ds, order, K), (ds, order, 1)])
        for sid, k in zip(ids, (K, 1)):
            epi.epi_wait(cx.ctx, sid)
            c, s, t = epi.epi_results(cx.ctx, sid, k, order)
            assert np.array_equal(c, r["combos"][:k]) and np.array_equal(s, r["scores"][:k])
            assert np.array_equal(t, r["tables"][:k])
            epi.epi_release(cx.ctx, sid)
    finally:
        epi.epi_unload(cx.ctx, ds)


@pytest.mark.parametrize("M,block", [(999, 4), (1000, 16), (1025, 16)])
def test_order2_default_kernel(cx, M, block):
    """The untuned order-2 kernel on both sides of its line, against the other
    one (the same integers, so the same results)."""
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(M, 321, seed=M, case_fraction=0.4)
    ds = cx.load(G, y)
    try:
        r = cx.scan(ds, 2, 40)
        assert r["prefix_block"] == block
        epi.epi_set_prefix_block(cx.ctx, ds, 2, 20 - block)
        o = cx.scan(ds, 2, 40)
        assert o["prefix_block"] == 20 - block
        for k in ("combos", "scores", "tables"):
            assert np.array_equal(r[k], o[k])
    finally:
        epi.epi_set_prefix_block(cx.ctx, ds, 2, 0)
        epi.epi_unload(cx.ctx, ds)
