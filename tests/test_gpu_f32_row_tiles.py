"""FP32 forward in tiles of 48 rows (8,193 to 12,288 sites of at most 64 outputs, or 512 tiles): four and eight
waves, one to four output blocks, whole, vector and word access, at the edges of that range; against float64
sums over the same neighbour map.  Tolerance as for the 16-row tiles: 2 N 2^-24 sum |x||w| for N products."""
import pytest
import torch

import paper_2509_24677_amd as npvs
from test_gpu_f32_matrix import DEV, padded, rows, rulebook

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sites,cin,cout", [
    (9000, 256, 64), (9000, 272, 48), (9000, 256, 32), (9000, 288, 16),  # eight waves
    (9000, 32, 32), (9000, 16, 48), (9000, 20, 64), (9000, 12, 32), (9000, 36, 24), (9000, 20, 12),  # whole, vector
    (9000, 27, 7), (9000, 3, 33), (9000, 5, 17), (9000, 19, 50), (9000, 264, 50), (9000, 257, 64),  # words
    (8192, 16, 64), (8193, 256, 48), (12288, 16, 33), (12289, 16, 48), (24576, 8, 64), (24577, 256, 16)])
def test_rows_of_48(sites, cin, cout):
    rb, nbr = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin * 1000 + cout)
    X = rows(sites, cin, rb.cap, gen)
    W = torch.randn((27, cin, cout), generator=gen, device=DEV)
    b = torch.randn(cout, generator=gen, device=DEV)
    Xz, idx = padded(X, sites), torch.where(nbr < 0, sites, nbr)
    ref = b.double().expand(sites, -1).clone()
    mag = b.double().abs().expand(sites, -1).clone()
    for k in range(27):
        ref += Xz[idx[k]] @ W[k].double()
        mag += Xz[idx[k]].abs() @ W[k].double().abs()
    out = torch.full((rb.cap, cout), float("nan"), device=DEV)
    npvs.sparse_conv_fwd(X, npvs.pack_weights(W, npvs.NPVS_F32), b, cin, cout, rb, npvs.NPVS_F32, False, out=out)
    err = (out[:sites].double() - ref).abs()
    assert bool((err <= 2 * (27 * cin + 2) * 2.0 ** -24 * mag).all()), float((err / mag).max())
    assert bool(torch.isnan(out[sites:]).all())
