"""Culling at the sizes where the triangles a workgroup takes change, over whole-word grids, ragged
grids and a PVS that is not 4-byte aligned: bit for bit the oracle's flags."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_24677_amd as npvs
from gpu_util import DEV, to_np, upload_tris
from test_gpu_cull import _adversarial, _pack, _random_pvs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,shift", [([(64, 24, 16), (32, 32, 32)], 0), ([(64, 24, 16), (32, 32, 32)], 1),
                                        ([(72, 24, 16), (32, 32, 32)], 0)])
def test_triangles_per_workgroup(dims, shift):
    rng = np.random.default_rng(7)
    base = [_adversarial(rng, 331, g) for g in dims]
    packed = [_pack(b) for b in _random_pvs(rng, dims, 0.02)]
    want = [oracle.visible_triangles(t, g, x) for t, g, x in zip(base, dims, packed)]
    assert all(0 < w.sum() < len(w) for w in want)
    flat = np.concatenate([np.zeros(shift, np.uint8)] + [x.reshape(-1) for x in packed])
    pvs = torch.from_numpy(flat).to(DEV)[shift:]
    for total in (1, 15, 16, 17, 10000, 10001, 32768, 32769, 300000, 300001):
        n = [total - total // 3, total // 3]
        pick = [np.arange(k) % 331 for k in n]
        tris, counts = upload_tris([t[p] for t, p in zip(base, pick)])
        got = to_np(npvs.visible_triangles(tris, counts, dims, pvs))
        np.testing.assert_array_equal(got, np.concatenate([w[p] for w, p in zip(want, pick)]))
