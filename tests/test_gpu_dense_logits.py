"""De-interleaving with dense logits, four froxels a thread and by bytes (rows of odd width, unaligned
rows, d < 4): value for value a numpy scatter."""
import numpy as np
import pytest
import torch

import paper_2509_24677_amd as npvs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("d", [2, 4, 8, 16, 32])
@pytest.mark.parametrize("pad,shift", [(0, 0), (4, 0), (1, 0), (0, 1)])
def test_dense_logits(d, pad, shift):
    rng = np.random.default_rng(d)
    dims = [(96, 32, 64), (32, 64, 32)] + ([(40, 8, 16), (8, 8, 8)] if d <= 8 else [])
    vox = [rng.random((nz, ny, nx)) < 2.0 / d ** 3 for nx, ny, nz in dims]
    vox[0][:] |= rng.random(vox[0].shape) < 1e-4
    occ = torch.from_numpy(np.concatenate([np.packbits(v, axis=2, bitorder="little").ravel() for v in vox])).to(DEV)
    rb = npvs.build_rulebook(occ, dims, d)
    n, C = int(rb.counts[0]), d ** 3
    y = rng.standard_normal((n, C + pad)).astype(np.float32)
    y[rng.random(y.shape) < 0.1] = 0.0
    y[rng.random(y.shape) < 0.02] = np.nan
    flat = torch.empty(rb.cap * (C + pad) + shift, dtype=torch.float32, device=DEV)
    Y = flat[shift:].view(rb.cap, C + pad)
    Y[:n] = torch.from_numpy(y).to(DEV)
    pvs, logits = npvs.deinterleave_threshold(Y, rb, occ, want_logits=True)
    bits, _ = npvs.deinterleave_threshold(Y, rb, occ)
    want_l, want_b, row = [], [], 0
    for v, (nx, ny, nz) in zip(vox, dims):
        act = v.reshape(nz // d, d, ny // d, d, nx // d, d).any(axis=(1, 3, 5))
        out = np.full((*act.shape, C), -np.inf, np.float32)
        k = int(act.sum())
        out[act] = y[row:row + k, :C]
        row += k
        out = out.reshape(nz // d, ny // d, nx // d, d, d, d).transpose(0, 3, 1, 4, 2, 5).reshape(nz, ny, nx)
        want_l.append(out.ravel())
        want_b.append(np.packbits((out >= 0) & v, axis=2, bitorder="little").ravel())
    assert row == n > 0
    np.testing.assert_array_equal(logits.cpu().numpy(), np.concatenate(want_l))
    np.testing.assert_array_equal(pvs.cpu().numpy(), np.concatenate(want_b))
    assert torch.equal(pvs, bits)
