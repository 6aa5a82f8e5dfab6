"""The largest counts of the kernels that hold both classes of a cell in one
float accumulator (needs an MI355X): panels with SNPs of a single genotype,
whose cells hold a whole class, at the class sizes where the packed sum comes
to the last integer below 2^24 (2047 individuals a class at four per count,
4095 at one), one step past the change between the two, and with one tiny
class.  Every combination is returned and compared with the oracle."""
from __future__ import annotations

import math

import numpy as np
import pytest

from parity import check_topk
from synth import random_genotypes

pytestmark = pytest.mark.gpu
MATRIX4, CROSS = 9, 8  # kernel variants


@pytest.fixture(scope="module")
def cx():
    from paper_2201_02460_amd import epi

    with epi.Context(0) as c:
        yield c


@pytest.mark.parametrize("order,M,n_cases,n_controls", [
    (4, 10, 2047, 2047), (4, 10, 1, 8190),
    (5, 9, 2047, 2047), (5, 9, 2048, 2048), (5, 10, 4095, 4095), (5, 9, 1, 16384),
    (6, 9, 4095, 4095), (6, 9, 16000, 385), (7, 10, 4095, 4095), (8, 10, 2047, 2047), (8, 10, 4095, 4095),
])
def test_whole_class_cells(cx, orc, order, M, n_cases, n_controls):
    from paper_2201_02460_amd import epi

    N = n_cases + n_controls
    G, y = random_genotypes(M, N, seed=N + order, case_fraction=n_cases / N)
    assert int(y.sum()) == n_cases
    # single-genotype SNPs, `order` of them: some combination has no other
    at = np.linspace(0, M - 1, order).astype(int)
    G[at] = (np.arange(order) % 3)[:, None].astype(G.dtype)
    print("case", order, M, n_cases, n_controls, flush=True)
    ds = cx.load(G, y)
    try:
        r = cx.scan(ds, order, 256)
        assert r["variant"] == (MATRIX4 if order == 4 else CROSS)
        assert len(r["combos"]) == math.comb(M, order)
        check_topk(orc, G, y, order, 256, r["combos"], r["scores"], r["tables"])
        sid = epi.epi_scan_check(cx.ctx, ds, order, 5)
        epi.epi_wait(cx.ctx, sid)
        assert epi.epi_scan_digest(cx.ctx, sid) == orc.digest(G, y, order)
        epi.epi_release(cx.ctx, sid)
    finally:
        epi.epi_unload(cx.ctx, ds)
