"""Froxelization where the binning's tables fill and its searches end: triangles scattered over more
tiles than a workgroup's table holds, triangles of more tiles than a thread remembers, and batches at
the edges of the grid search.  Bit for bit the oracle; the rulebook of each batch as the union of its
grids' own."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_24677_amd as npvs
from gpu_util import to_np, upload_tris

pytestmark = pytest.mark.gpu


def scattered(rng, n, dims, size):
    c = rng.uniform(0, np.array(dims, np.float64), size=(n, 1, 3))
    return (c + rng.uniform(-size, size, size=(n, 3, 3))).astype(np.float32)


@pytest.mark.parametrize("grids", [1, 2, 7, 8, 9, 17, 32])
@pytest.mark.parametrize("size", [0.5, 12.0])  # one tile mostly; up to dozens
def test_bins_and_grid_search(grids, size):
    rng = np.random.default_rng(grids)
    dims = [[(256, 128, 128), (32, 40, 16), (64, 8, 72)][i % 3] if grids > 1 else (256, 256, 128) for i in range(grids)]
    n = [0 if i == 1 and grids > 2 else 700 if g[0] == 256 else 60 for i, g in enumerate(dims)]
    tri_list = [scattered(rng, k, g, size) for k, g in zip(n, dims)]
    tris, counts = upload_tris(tri_list)
    occ = npvs.froxelize(tris, counts, dims)
    want = [oracle.froxelize(t, g)[0].ravel() for t, g in zip(tri_list, dims)]
    np.testing.assert_array_equal(to_np(occ), np.concatenate(want))
    rb = npvs.build_rulebook(occ, dims, 8)
    row = 0
    for b, (w, g) in enumerate(zip(want, dims)):  # each grid by itself: rows, table and neighbours moved by the rows before
        one = npvs.build_rulebook(torch.from_numpy(w).to(occ.device), [g], 8)
        k = int(one.counts[0])
        nbr = to_np(one.nbr[:, :k])
        np.testing.assert_array_equal(to_np(rb.nbr[:, row:row + k]), np.where(nbr >= 0, nbr + row, -1))
        assert int(rb.grid_rows[b]) == row
        row += k
    assert int(rb.counts[0]) == row
