"""Site tables, neighbour maps and pair lists at the edges of their vector paths
(blocks per thread, rows per workgroup and per pair count, alignment, capacity), integer for integer
against numpy."""
import numpy as np
import pytest
import torch

import paper_2509_24677_amd as npvs

pytestmark = pytest.mark.gpu
DEV = "cuda"


def reference(vox, dims, d, cap):
    """Sites needed, site keys, block_row, grid_rows, nbr and pairs."""
    act, offs = [], [0]
    for v, (nx, ny, nz) in zip(vox, dims):
        b = v.reshape(nz // d, d, ny // d, d, nx // d, d).transpose(0, 2, 4, 1, 3, 5).reshape(-1, d ** 3)
        act.append(b.any(1))
        offs.append(offs[-1] + len(b))
    act = np.concatenate(act)
    keys = np.nonzero(act)[0][:cap]
    row = np.full(len(act), -1, np.int64)
    row[keys] = np.arange(len(keys))
    nbr = np.full((27, len(keys)), -1, np.int64)
    for g, (nx, ny, nz) in enumerate(dims):
        r = np.nonzero((keys >= offs[g]) & (keys < offs[g + 1]))[0]
        n = np.array([nx, ny, nz]) // d
        pos = np.stack(np.unravel_index(keys[r] - offs[g], n[::-1])[::-1], 1)
        for k in range(27):
            q = pos + [k % 3 - 1, k // 3 % 3 - 1, k // 9 - 1]
            ok = ((q >= 0) & (q < n)).all(1)
            q = q[ok]
            nbr[k, r[ok]] = row[offs[g] + (q[:, 2] * n[1] + q[:, 1]) * n[0] + q[:, 0]]
    pairs = np.concatenate([np.stack([nbr[k][nbr[k] >= 0], np.nonzero(nbr[k] >= 0)[0]], 1) for k in range(27)])
    return int(act.sum()), keys, row, np.searchsorted(keys, offs), nbr, pairs


@pytest.mark.parametrize("d,density", [(1, 0.4), (2, 0.1), (4, 0.02), (8, 0.004), (16, 0.002), (32, 1e-4), (4, 0.0)])
@pytest.mark.parametrize("wide", [True, False])  # every nx a multiple of 32, or not
def test_site_tables(d, density, wide):
    rng = np.random.default_rng(d)
    dims = [(32, 32, 32), (64, 32, 96), (32, 96, 32)]
    if not wide and d < 32:
        dims[1] = (48, 32, 64) if d > 8 else (40, 32, 64)
    vox = [rng.random((nz, ny, nx)) < density for nx, ny, nz in dims]
    packed = np.concatenate([np.packbits(v, axis=2, bitorder="little").ravel() for v in vox])
    occ = torch.from_numpy(packed).to(DEV)
    total = reference(vox, dims, d, 1 << 30)[0]
    for cap in (None, max(total // 2, 1)):
        want = reference(vox, dims, d, cap or 1 << 30)
        for shift in (0, 1):  # 1: a site table that is not 16-byte aligned
            rb = npvs.build_rulebook(occ, dims, d, cap=cap, csr=True)
            rb.block_row = torch.empty(rb.block_row.numel() + shift, dtype=torch.int32, device=DEV)[shift:]
            rb = npvs.build_rulebook(occ, dims, d, cap=rb.cap, csr=True, out=rb)
            n = len(want[1])
            counts = rb.counts.cpu().numpy()
            assert counts[0] == n and counts[1] == want[0]
            assert np.array_equal(rb.site_keys[:n].cpu().numpy(), want[1])
            assert np.array_equal(rb.block_row.cpu().numpy(), want[2])
            assert np.array_equal(rb.grid_rows.cpu().numpy(), want[3])
            assert np.array_equal(rb.nbr[:, :n].cpu().numpy(), want[4])
            assert np.array_equal(rb.rb_pairs[:len(want[5])].cpu().numpy(), want[5])
            off = np.concatenate([[0], np.cumsum((want[4] >= 0).sum(1))])
            assert np.array_equal(rb.rb_off.cpu().numpy(), off)
