"""The staged BF16 shape in its steady state and at the edge of it: a workgroup walks tiles of 16 rows (256
workgroups), fetches indices six tiles ahead into a ring of eight slots, and only from seven tiles on
takes them from there; three or four output blocks.  Bit for bit the single-role shape, which sums the
same products in the same order."""
import pytest
import torch

import paper_2509_24677_amd as npvs
from test_gpu_f32_matrix import rows, rulebook

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("sites", [17, 4097, 24575, 24576, 24577, 28673, 32769, 45057, 60000])  # 1 to 15 tiles
@pytest.mark.parametrize("cin,cout", [(8, 40), (32, 48), (8, 64), (24, 56), (40, 8), (40, 64), (64, 48), (64, 64)])
def test_many_tiles(sites, cin, cout):
    rb, _ = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin * 100 + cout)
    X = rows(sites, cin, rb.cap, gen).to(torch.bfloat16)  # rows past the sites NaN: never read
    Wp = npvs.pack_weights(torch.randn((27, cin, cout), generator=gen, device=DEV), npvs.NPVS_BF16)
    b = torch.randn(cout, generator=gen, device=DEV)
    for bias, relu, f32 in ((b, True, False), (None, False, True)):
        out = [torch.full((rb.cap, cout), float("nan"), dtype=torch.float32 if f32 else torch.bfloat16, device=DEV)
               for _ in range(2)]
        got, want = (npvs.sparse_conv_fwd(X, Wp, bias, cin, cout, rb, npvs.NPVS_BF16, relu, out_f32=f32, variant=v,
                                          out=o) for v, o in zip((None, 14), out))
        assert bool(torch.isfinite(want[:sites].float()).all())
        assert torch.equal(got[:sites], want[:sites])
        assert bool(torch.isnan(got[sites:].float()).all())  # rows past the sites: not written
