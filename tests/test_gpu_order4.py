"""Order 4 on the matrix cores (needs an MI355X): the edges of its item blocks
(32 first SNPs, 16 last ones) and of its operand rows (classes around
multiples of 96 individuals), its rule, and scans over several blocks, against
the oracle and the all-cell kernel."""
from __future__ import annotations

import math

import numpy as np
import pytest

from parity import check_topk
from synth import random_genotypes

pytestmark = pytest.mark.gpu
MATRIX, POPCOUNT = 9, 5  # kernel variants


@pytest.fixture(scope="module")
def cx():
    from paper_2201_02460_amd import epi

    with epi.Context(0) as c:
        yield c


@pytest.mark.parametrize("M,N,n_cases,K", [
    (4, 40, 20, 1), (5, 97, 96, 5), (15, 193, 97, 30), (16, 288, 192, 256), (17, 385, 96, 40), (18, 96, 95, 7),
    (31, 291, 98, 20), (32, 200, 100, 50),
])
def test_order4_block_edges(cx, orc, M, N, n_cases, K):
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(M, N, seed=41 * M + N, case_fraction=n_cases / N)
    print("case", M, N, K, flush=True)
    ds = cx.load(G, y)
    try:
        r = cx.scan(ds, 4, K)
        assert r["variant"] == MATRIX and len(r["combos"]) == min(K, math.comb(M, 4))
        check_topk(orc, G, y, 4, K, r["combos"], r["scores"], r["tables"])
        sid = epi.epi_scan_check(cx.ctx, ds, 4, K)
        epi.epi_wait(cx.ctx, sid)
        assert epi.epi_scan_digest(cx.ctx, sid) == orc.digest(G, y, 4)
        epi.epi_release(cx.ctx, sid)
        ids = epi.epi_scan_batch(cx.ctx, [(ds, 4, K), (ds, 2, 3)])  # beside another order, in a graph
        epi.epi_wait(cx.ctx, ids[0])
        for a, b in zip(epi.epi_results(cx.ctx, ids[0], K, 4), (r["combos"], r["scores"], r["tables"])):
            assert np.array_equal(a, b)
        for sid in ids:
            epi.epi_release(cx.ctx, sid)
    finally:
        epi.epi_unload(cx.ctx, ds)


@pytest.mark.parametrize("M,N,n_cases,variant", [
    (83, 4000, 2000, MATRIX), (115, 2001, 600, MATRIX), (82, 4000, 2000, POPCOUNT), (115, 1999, 600, POPCOUNT),
    (33, 500, 250, POPCOUNT), (20, 8191, 400, MATRIX), (20, 8192, 400, POPCOUNT), (20, 4200, 2100, POPCOUNT),
])
def test_order4_rule_and_digest(cx, M, N, n_cases, variant):
    """Every combination once, each with its table, as the all-cell kernel."""
    from paper_2201_02460_amd import epi

    G, y = random_genotypes(M, N, seed=M + N, case_fraction=n_cases / N)
    ds = cx.load(G, y)
    got = []
    try:
        for block in (0, epi.EPI_BLOCK_ALL_CELLS):
            print("case", M, N, n_cases, "block", block, flush=True)
            epi.epi_set_prefix_block(cx.ctx, ds, 4, block)
            sid = epi.epi_scan_check(cx.ctx, ds, 4, 10)
            epi.epi_wait(cx.ctx, sid)
            if block == 0:
                assert epi.epi_scan_info(cx.ctx, sid)["variant"] == variant
            res = epi.epi_results(cx.ctx, sid, 10, 4)
            got.append((epi.epi_scan_digest(cx.ctx, sid), [x.tolist() for x in res]))
            epi.epi_release(cx.ctx, sid)
        assert got[0][0][0] == math.comb(M, 4)
        assert got[0] == got[1]
    finally:
        epi.epi_set_prefix_block(cx.ctx, ds, 4, 0)
        epi.epi_unload(cx.ctx, ds)
