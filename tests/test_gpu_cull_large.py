"""Culling around 65,536 triangles, where workgroups take 64 with half the threads, and above 524,288, where
they take several groups each: bit for bit the oracle's flags; with triangles outside every grid among them."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_24677_amd as npvs
from gpu_util import DEV, to_np, upload_tris
from test_gpu_cull import _adversarial, _pack, _random_pvs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("total", [65535, 65536, 65537, 65600, 130001, 524289, 600000])
@pytest.mark.parametrize("nx", [64, 72])  # whole PVS words, or bytes
def test_large_totals(total, nx):
    dims = [(nx, 24, 16), (32, 32, 32)]
    rng = np.random.default_rng(total)
    base = [_adversarial(rng, 331, g) for g in dims]
    for t in base:
        t[::3] += 300.0
    packed = [_pack(b) for b in _random_pvs(rng, dims, 0.02)]
    want = [oracle.visible_triangles(t, g, x) for t, g, x in zip(base, dims, packed)]
    assert all(0 < w.sum() < len(w) for w in want)
    pvs = torch.from_numpy(np.concatenate([x.reshape(-1) for x in packed])).to(DEV)
    n = [total - total // 3, total // 3]
    pick = [np.arange(k) % 331 for k in n]
    tris, counts = upload_tris([t[p] for t, p in zip(base, pick)])
    got = to_np(npvs.visible_triangles(tris, counts, dims, pvs))
    np.testing.assert_array_equal(got, np.concatenate([w[p] for w, p in zip(want, pick)]))
