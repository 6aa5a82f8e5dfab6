"""Persistent batches of several scans of one order from 4 up, over datasets
of different sizes (needs an MI355X): a workgroup's run of work items crosses
from one scan into the next, whose items need the next dataset's screening
table.  Small panels are asked for every combination (none may be missing);
larger ones must return what their plain scans return, over replays."""
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


def load(cx, shapes, seed):
    data = [random_genotypes(M, N, seed=seed + i, case_fraction=f) for i, (M, N, f) in enumerate(shapes)]
    return data, [cx.load(G, y) for G, y in data]


# item counts per scan: order 4 21, 15, 28; 5 14, 11, 24; 6 18, 8, 38; 7 22, 6, 63; 8 9, 45, 165
@pytest.mark.parametrize("order,panels", [(4, (9, 8, 10)), (5, (9, 8, 10)), (6, (9, 8, 10)), (7, (9, 8, 10)),
                                          (8, (9, 10, 11))])
def test_batch_returns_every_combination(cx, orc, order, panels):
    from paper_2201_02460_amd import epi

    shapes = [(M, N, f) for M, N, f in zip(panels, (130, 301, 97), (0.4, 0.5, 0.3))]
    data, dss = load(cx, shapes, 100 * order)
    K = 256
    try:
        print("case", order, panels, flush=True)
        ids = epi.epi_scan_batch(cx.ctx, [(ds, order, K) for ds in dss])
        for sid, (G, y) in zip(ids, data):
            epi.epi_wait(cx.ctx, sid)
            c, s, t = epi.epi_results(cx.ctx, sid, K, order)
            assert len(c) == math.comb(G.shape[0], order)
            check_topk(orc, G, y, order, K, c, s, t)
            epi.epi_release(cx.ctx, sid)
    finally:
        for ds in dss:
            epi.epi_unload(cx.ctx, ds)


@pytest.mark.parametrize("order,panels", [(4, (31, 25, 18, 32)), (5, (21, 17, 25)), (6, (15, 18, 13)), (7, (13, 12, 14)),
                                          (8, (12, 11, 13))])
@pytest.mark.parametrize("use_graph", [False, True])
def test_batch_equals_plain_scans(cx, order, panels, use_graph):
    from paper_2201_02460_amd import epi

    shapes = [(M, 150 + 77 * i + 5 * M, 0.35 + 0.05 * i) for i, M in enumerate(panels)]
    _, dss = load(cx, shapes, 200 * order)
    Ks = [40, 7, 200, 1]
    descs = [(ds, order, K) for ds, K in zip(dss, Ks)]
    try:
        print("case", order, panels, use_graph, flush=True)
        plain = [cx.scan(ds, o, K) for ds, o, K in descs]
        bid = epi.epi_batch_create(cx.ctx, descs, persistent=True, use_graph=use_graph)
        for rep in range(3):
            epi.epi_batch_run(cx.ctx, bid)
            epi.epi_batch_wait(cx.ctx, bid)
            for i, (_, o, K) in enumerate(descs):
                got = epi.epi_batch_results(cx.ctx, bid, i, K, o)
                for a, b in zip(got, (plain[i]["combos"], plain[i]["scores"], plain[i]["tables"])):
                    assert np.array_equal(a, b), f"replay {rep}, scan {i}"
        epi.epi_batch_destroy(cx.ctx, bid)
    finally:
        for ds in dss:
            epi.epi_unload(cx.ctx, ds)
