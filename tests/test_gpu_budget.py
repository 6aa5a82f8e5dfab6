"""Scans and batches of orders 4-8 under tight memory budgets (needs an
MI355X): whatever fits with the popcount kernel pinned is accepted with the
built-in choice too and returns the same, from budgets that hold nothing but
the popcount scan to budgets with room for the matrix-core kernels' cell rows
and larger launches."""
from __future__ import annotations

import numpy as np
import pytest

from synth import random_genotypes

pytestmark = pytest.mark.gpu
CROSS, REDUCED_MATRIX, REDUCED, POPCOUNT = 8, 9, 5, 0  # kernel variants
K = 256


def run(budget, data, scans, pin, batch):
    """Results and variants of the scans (dataset index, order) in a context of
    `budget` bytes; None if it refuses them for lack of memory."""
    from paper_2201_02460_amd import epi

    with epi.Context(0, budget) as cx:
        try:
            dss = [cx.load(G, y) for G, y in data]
            for d, o in scans if pin else ():
                epi.epi_set_prefix_block(cx.ctx, dss[d], o, epi.EPI_BLOCK_ALL_CELLS)
            descs = [(dss[d], o, K) for d, o in scans]
            ids = epi.epi_scan_batch(cx.ctx, descs) if batch else [epi.epi_scan(cx.ctx, *descs[0])]
        except epi.EpiError as e:
            assert e.code == epi.EPI_ENOMEM
            return None
        out = []
        for sid, (_, o, k) in zip(ids, descs):
            epi.epi_wait(cx.ctx, sid)
            out.append((epi.epi_scan_info(cx.ctx, sid)["variant"], epi.epi_results(cx.ctx, sid, k, o)))
            epi.epi_release(cx.ctx, sid)
        return out


def used_by(data):
    from paper_2201_02460_amd import epi

    with epi.Context(0) as cx:
        for G, y in data:
            cx.load(G, y)
        return epi.epi_memory(cx.ctx)[0]


@pytest.mark.parametrize("shapes,scans,batch", [
    ([(20, 1000)], [(0, 5)], False),
    # one set of rows for the scans of a dataset, and another dataset's
    ([(20, 1000), (18, 900)], [(0, 5), (0, 5), (1, 5), (0, 6), (1, 5)], True),
])
def test_budget_accepts_what_popcount_fits(shapes, scans, batch):
    data = [random_genotypes(M, N, seed=M + N, case_fraction=0.45) for M, N in shapes]
    base = used_by(data)
    room, variants = 1 << 20, []
    while not variants or set(variants[-1]) != {CROSS}:
        assert room < 1 << 28
        room += room // 16
        p = run(base + room, data, scans, True, batch)
        if p is None:
            continue
        got = run(base + room, data, scans, False, batch)
        print("room", room, "variants", None if got is None else [v for v, _ in got], flush=True)
        assert got is not None, "refused with room for the popcount kernel"
        for (_, r), (_, w) in zip(got, p):
            for a, b in zip(r, w):
                assert np.array_equal(a, b)
        variants.append([v for v, _ in got])
    assert set(variants[0]) == {POPCOUNT}


def test_budget_order4():
    """Order 4: the reduced-cell kernel on the vector units where the
    matrix-core one's launch does not fit."""
    data = [random_genotypes(31, 700, seed=4, case_fraction=0.45)]
    base = used_by(data)
    want = run(0, data, [(0, 4)], False, False)[0]
    room, seen = 1 << 18, []
    while not seen or seen[-1] != REDUCED_MATRIX:
        assert room < 1 << 28
        room += room // 16
        got = run(base + room, data, [(0, 4)], False, False)
        print("room", room, "variant", None if got is None else got[0][0], flush=True)
        if got is None:
            assert not seen, "refused with more room than an accepted scan had"
            continue
        for a, b in zip(got[0][1], want[1]):
            assert np.array_equal(a, b)
        seen.append(got[0][0])
    assert seen[0] == REDUCED
