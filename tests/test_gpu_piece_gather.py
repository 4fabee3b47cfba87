"""512 inputs, gathered by 64-byte pieces, against the general kernel's 32-row shape at the edges of its
tiles: the same products, summed chunk by chunk within nine groups of offsets, bit for bit."""
import pytest
import torch

import paper_2509_24677_amd as npvs
from test_gpu_f32_matrix import rows, rulebook

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("sites", [1, 15, 16, 17, 31, 33, 300, 1802])
@pytest.mark.parametrize("cin", [488, 512])
@pytest.mark.parametrize("cout", [56, 64])
def test_pieces_of_wide_rows(sites, cin, cout):
    rb, _ = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin + cout)
    X = rows(sites, cin, rb.cap, gen).to(torch.bfloat16)  # rows past the sites NaN: never read
    W = torch.randn((27, cin, cout), generator=gen, device=DEV)
    b = torch.randn(cout, generator=gen, device=DEV)
    got, two = (npvs.sparse_conv_fwd(X, npvs.pack_weights(W, npvs.NPVS_BF16), b, cin, cout, rb, npvs.NPVS_BF16, True,
                                     out_f32=True, variant=v) for v in (None, 5))
    # 72 outputs go through the general kernel, whose first outputs have the same weights
    W2, b2 = torch.zeros((27, cin, 72), device=DEV), torch.zeros(72, device=DEV)
    W2[..., :cout], b2[:cout] = W, b
    want = npvs.sparse_conv_fwd(X, npvs.pack_weights(W2, npvs.NPVS_BF16), b2, cin, 72, rb, npvs.NPVS_BF16, True,
                                out_f32=True)
    assert bool(torch.isfinite(want[:sites]).all())
    assert torch.equal(got[:sites], want[:sites, :cout])
    assert torch.equal(two[:sites], want[:sites, :cout])
