"""Contingency tables and mutual information of listed combinations (needs an
MI355X) at the edges of a wave's 64 combinations and of the halves its tables
are stored by, against counts and entropies in numpy; invalid combinations
among valid ones leave their tables unwritten."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cx():
    from paper_2201_02460_amd import epi

    with epi.Context(0) as c:
        yield c


def xlogx(n):
    n = np.asarray(n, dtype=np.float64)
    return np.where(n > 0, n * np.log(np.maximum(n, 1)), 0.0)


@pytest.mark.parametrize("order", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("n", [1, 31, 33, 63, 64, 65, 160])
def test_tables_edges(cx, order, n):
    import torch

    from paper_2201_02460_amd import epi

    M, N, P = 14, 131 + n, 3**order
    rng = np.random.default_rng(100 * order + n)
    G = rng.integers(0, 3, (M, N)).astype(np.uint8)
    y = (rng.random(N) < 0.4).astype(np.uint8)
    combos = np.sort(np.argsort(rng.random((n, M)), axis=1)[:, :order], axis=1).astype(np.int32)
    print("case", order, n, flush=True)
    cell = np.zeros((n, N), np.int64)
    for t in range(order):
        cell = 3 * cell + G[combos[:, t]]
    want = np.stack([np.stack([np.bincount(cell[i][y == c], minlength=P) for c in (1, 0)]) for i in range(n)])
    ds = cx.load(G, y)
    try:
        # one word past the tables stays as it was
        flat = torch.full((n * 2 * P + 1,), 77, dtype=torch.int32, device="cuda")
        tabs = flat[:-1].view(n, 2, P)
        epi.epi_contingency_tables(cx.ctx, ds, torch.from_numpy(combos).cuda(), tabs)
        assert np.array_equal(tabs.cpu().numpy(), want) and int(flat[-1]) == 77
        mi = torch.zeros(n, dtype=torch.float64, device="cuda")
        epi.epi_mutual_information(cx.ctx, ds, order, tabs, mi)
        nc = np.array([y.sum(), N - y.sum()])
        ref = (xlogx(want).sum((1, 2)) - xlogx(want.sum(1)).sum(1) - xlogx(nc).sum() + xlogx(N)) / N
        # terms of 3 rounded table entries a cell, 2^-35 at least, and the sums in float64
        assert np.abs(mi.cpu().numpy() - ref).max() <= (3 * P + 3) * 2.0**-35 / N + 1e-12
        # an index out of range: an error, its own table unwritten, the others written
        bad = combos.copy()
        bad[n // 2, 0] = M
        flat.fill_(77)
        with pytest.raises(epi.EpiError):
            epi.epi_contingency_tables(cx.ctx, ds, torch.from_numpy(bad).cuda(), tabs)
        want[n // 2] = 77
        assert np.array_equal(tabs.cpu().numpy(), want)
    finally:
        epi.epi_unload(cx.ctx, ds)
