"""The default BF16 shape (rows staged through LDS, partial sums added by reducer waves) at the edges
of its tiles and channel counts: bit for bit the single-role weight-stationary shape, which sums the
same products in the same order."""
import pytest
import torch

import paper_2509_24677_amd as npvs
from test_gpu_f32_matrix import rows, rulebook

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("sites", [1, 15, 16, 17, 300, 4097, 20000])
@pytest.mark.parametrize("cin,cout", [(8, 8), (16, 64), (24, 40), (32, 16), (40, 64), (64, 24), (64, 64)])
def test_staged_equals_single_role(sites, cin, cout):
    rb, _ = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin * 100 + cout)
    X = rows(sites, cin, rb.cap, gen).to(torch.bfloat16)  # rows past the sites NaN: never read
    Wp = npvs.pack_weights(torch.randn((27, cin, cout), generator=gen, device=DEV), npvs.NPVS_BF16)
    b = torch.randn(cout, generator=gen, device=DEV)
    for bias, relu, f32 in ((b, True, False), (None, False, True)):
        got, want = (npvs.sparse_conv_fwd(X, Wp, bias, cin, cout, rb, npvs.NPVS_BF16, relu, out_f32=f32, variant=v)
                     for v in (None, 14))
        assert bool(torch.isfinite(want[:sites].float()).all())
        assert torch.equal(got[:sites], want[:sites])
