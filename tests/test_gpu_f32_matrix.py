"""FP32 layers on the matrix cores at the edges of their tiles: forward and data gradient (row
tiles of 16 and 48, channel substeps of 16, output blocks of 16, vector and word access) and weight
gradient (chunks of 32 pairs, products of 4, narrow and ragged windows), against float64 sums over
the same neighbour map.

Tolerances: a float32 sum of N products in any order is within gamma_N sum |x||w| of the exact one;
2 N 2^-24 covers it with the rounding of the result.  A weight-gradient entry is a compensated sum
of plain sums of at most 32 products: 2 * 40 * 2^-24 sum |x||dz|."""
import numpy as np
import pytest
import torch

import paper_2509_24677_amd as npvs

pytestmark = pytest.mark.gpu
DEV = "cuda"


def rulebook(sites, seed, csr=False):
    """A rulebook of `sites` active blocks (d = 4) clustered in the low corner of a grid."""
    side = 8
    while side ** 3 < 3 * sites:
        side += 8
    g = np.random.default_rng(seed)
    m = np.zeros((side, side, side), bool)
    flat = m.reshape(-1)
    flat[g.choice(min(3 * sites, flat.size), sites, replace=False)] = True
    v = np.zeros((4 * side, 4 * side, 4 * side), bool)
    v[::4, ::4, ::4] = m
    bits = torch.from_numpy(np.packbits(v, axis=-1, bitorder="little").reshape(-1)).to(DEV)
    rb = npvs.build_rulebook(bits, [(4 * side,) * 3], 4, csr=csr)
    assert rb.host_counts()["n_sites"] == sites
    return rb, rb.nbr[:, :sites].long()


def rows(n, c, cap, gen, offset=0):
    """[cap][c] float32 with n random rows, the rest NaN (never read); `offset` floats past an
    aligned address."""
    buf = torch.full((cap * c + offset,), float("nan"), device=DEV)
    t = buf[offset:].view(cap, c)
    t[:n] = torch.randn((n, c), generator=gen, device=DEV)
    return t


def padded(t, n):
    return torch.cat([t[:n].double(), torch.zeros((1, t.shape[1]), dtype=torch.float64, device=DEV)])


@pytest.mark.parametrize("sites,cin,cout,offset", [
    (1, 64, 64, 0), (15, 8, 16, 0), (17, 16, 48, 0), (47, 64, 80, 0), (49, 27, 33, 0), (300, 1, 1, 0),
    (300, 3, 65, 0), (300, 64, 64, 1), (300, 12, 6, 0), (300, 256, 64, 0), (300, 260, 20, 0), (1000, 160, 96, 0),
    (4100, 64, 32, 0), (9699, 64, 64, 0), (24577, 8, 16, 0), (24577, 20, 64, 0)])
def test_conv_fwd_f32_tiles(sites, cin, cout, offset):
    rb, nbr = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin * 1000 + cout)
    X = rows(sites, cin, rb.cap, gen, offset)
    W = torch.randn((27, cin, cout), generator=gen, device=DEV)
    b = torch.randn(cout, generator=gen, device=DEV)
    Xz, idx = padded(X, sites), torch.where(nbr < 0, sites, nbr)
    ref = b.double().expand(sites, -1).clone()
    mag = b.double().abs().expand(sites, -1).clone()
    for k in range(27):
        ref += Xz[idx[k]] @ W[k].double()
        mag += Xz[idx[k]].abs() @ W[k].double().abs()
    for relu in (False, True):
        Y = npvs.sparse_conv_fwd(X, npvs.pack_weights(W, npvs.NPVS_F32), b, cin, cout, rb, npvs.NPVS_F32, relu)
        want = ref.clamp_min(0) if relu else ref
        err = (Y[:sites].double() - want).abs()
        assert bool((err <= 2 * (27 * cin + 2) * 2.0 ** -24 * mag).all()), float((err / mag).max())


@pytest.mark.parametrize("sites,cin,cout,offset", [
    (1, 64, 64, 0), (5, 8, 16, 0), (33, 16, 33, 0), (300, 1, 1, 0), (300, 3, 65, 0), (300, 64, 64, 1), (300, 17, 32, 0),
    (300, 50, 16, 0), (300, 130, 20, 0), (4100, 32, 64, 0), (9699, 64, 64, 0)])
def test_wgrad_f32_windows(sites, cin, cout, offset):
    rb, nbr = rulebook(sites, sites, csr=True)
    gen = torch.Generator(device=DEV).manual_seed(cin * 1000 + cout)
    X = rows(sites, cin, rb.cap, gen, offset)
    dY = rows(sites, cout, rb.cap, gen)
    W = torch.randn((27, cin, cout), generator=gen, device=DEV)
    _, dW, db = npvs.sparse_conv_bwd(X, npvs.pack_weights(W, npvs.NPVS_F32, True), cin, cout, None, dY, rb,
                                     npvs.NPVS_F32, False, want_dx=False)
    Xz, idx, dZ = padded(X, sites), torch.where(nbr < 0, sites, nbr), dY[:sites].double()
    for k in range(27):
        ref = Xz[idx[k]].T @ dZ
        mag = Xz[idx[k]].abs().T @ dZ.abs()
        err = (dW[k].double() - ref).abs()
        assert bool((err <= 80 * 2.0 ** -24 * mag).all()), (k, float((err / mag.clamp_min(1e-30)).max()))
