"""Packing (needs an MI355X): the rows of every SNP against the genotypes, at
the edges of a wave's SNPs (16) and individuals (64, 128) and of the class
index map's chunks (1024 individuals), and a repack in place."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cx():
    from paper_2201_02460_amd import epi

    with epi.Context(0) as c:
        yield c


def rows_of(G, y):
    """Bit rows [M, 3, words] of each genotype, cases first, each class padded to 128 individuals."""
    M, out = G.shape[0], []
    for cl in (1, 0):
        g = G[:, y == cl]
        pad = (-g.shape[1]) % 128
        g = np.pad(g, ((0, 0), (0, pad)), constant_values=3)
        bits = (g[:, None, :] == np.arange(3)[None, :, None]).astype(np.uint8)
        out.append(np.packbits(bits, axis=2, bitorder="little").view("<u4").reshape(M, 3, -1))
    return np.concatenate(out, axis=2)


@pytest.mark.parametrize("M,N,n_cases", [
    (2, 2, 1), (15, 63, 31), (16, 128, 64), (17, 129, 65), (33, 1023, 128), (63, 1024, 127), (64, 1025, 513),
    (65, 2049, 1024), (130, 3100, 129),
])
def test_packed_rows(cx, M, N, n_cases):
    import torch

    from paper_2201_02460_amd import epi

    rng = np.random.default_rng(M * N)
    print("case", M, N, n_cases, flush=True)
    ds = None
    try:
        for rep in range(2):  # the second time into the same dataset
            G = rng.integers(0, 3, (M, N)).astype(np.uint8)
            y = np.zeros(N, np.uint8)
            y[rng.permutation(N)[:n_cases]] = 1
            if ds is None:
                ds = cx.load(G, y)
            else:
                # rows with a stride, starting at any byte
                wide = torch.empty((M, N + 5), dtype=torch.uint8, device="cuda")
                g = wide[:, 3:3 + N]
                g.copy_(torch.from_numpy(G))
                epi.epi_repack_device(cx.ctx, ds, g, torch.from_numpy(y).cuda())
            want = rows_of(G, y)
            combos = torch.arange(M, dtype=torch.int32, device="cuda").reshape(M, 1)
            rows = torch.empty((M, 3, want.shape[2]), dtype=torch.int32, device="cuda")
            epi.epi_genotype_tables(cx.ctx, ds, combos, rows)
            torch.cuda.synchronize()
            assert np.array_equal(rows.cpu().numpy().view(np.uint32), want)
    finally:
        if ds is not None:
            epi.epi_unload(cx.ctx, ds)
