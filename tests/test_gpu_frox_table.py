"""Froxelization around the number of wide triangles at which a workgroup of the binning uses the whole of its
tile table: 256 triangles a workgroup, `wide` of them over many tiles, the rest over one or two; on grids
with and without whole output words.  Bit for bit the oracle."""
import numpy as np
import pytest

import oracle
import paper_2509_24677_amd as npvs
from gpu_util import to_np, upload_tris

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wide", [0, 1, 47, 48, 49, 200, 256])
@pytest.mark.parametrize("total", [255, 256, 700])
@pytest.mark.parametrize("nx", [256, 248])
def test_table_halves(wide, total, nx):
    rng = np.random.default_rng(wide * 1000 + total)
    dims = (nx, 128, 64)
    size = np.where(np.arange(total) % 256 < wide, 10.0, 0.4)[:, None, None]
    tri = (rng.uniform(0, dims, (total, 1, 3)) + rng.uniform(-1, 1, (total, 3, 3)) * size).astype(np.float32)
    order = np.concatenate([b + rng.permutation(min(256, total - b)) for b in range(0, total, 256)])
    tri = tri[order]  # anywhere among a workgroup's waves
    tris, counts = upload_tris([tri])
    np.testing.assert_array_equal(to_np(npvs.froxelize(tris, counts, [dims])).ravel(),
                                  oracle.froxelize(tri, dims)[0].ravel())
