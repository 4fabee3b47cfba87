"""The general BF16 kernel at the site counts where its rows per tile change, with and without input
ranges: every row written, bit for bit the 32-row shape, which sums the same products in the same
order, and within BF16's rounding of a float64 sum on a few rows."""
import pytest
import torch

import paper_2509_24677_amd as npvs
from test_gpu_f32_matrix import rows, rulebook

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("sites", [1, 16, 17, 65, 250, 400, 520, 1030, 2050, 4097])
@pytest.mark.parametrize("cin,cout", [(168, 72), (512, 96), (1024, 64), (1024, 136), (2056, 8)])
def test_rows_per_tile(sites, cin, cout):
    rb, _ = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin + cout)
    X = rows(sites, cin, rb.cap, gen).to(torch.bfloat16)  # rows past the sites NaN: never read
    W = torch.randn((27, cin, cout), generator=gen, device=DEV)
    Wp = npvs.pack_weights(W, npvs.NPVS_BF16)
    b = torch.randn(cout, generator=gen, device=DEV)
    got, want = (npvs.sparse_conv_fwd(X, Wp, b, cin, cout, rb, npvs.NPVS_BF16, False, out_f32=True, variant=v,
                                      out=torch.full((rb.cap, cout), float("nan"), device=DEV)) for v in (None, 5))
    assert torch.equal(got[:sites], want[:sites])
    assert bool(torch.isfinite(got[:sites]).all()) and bool(torch.isnan(got[sites:]).all())
    pick = torch.tensor(sorted({0, sites // 2, sites - 1}), device=DEV)
    ref = b.double().repeat(len(pick), 1)
    mag = torch.zeros_like(ref)
    Wd = W.to(torch.bfloat16).double()
    for k in range(27):
        i = rb.nbr[k, pick].long()
        x = torch.where((i >= 0)[:, None], X[i.clamp(min=0)].double(), torch.zeros((), dtype=torch.float64, device=DEV))
        ref += x @ Wd[k]
        mag += x.abs() @ Wd[k].abs()
    # float32 accumulation of 27 cin products: half an ulp of the running sum each, at most
    assert bool(((got[pick].double() - ref).abs() <= 27 * cin * 2.0 ** -24 * mag + 2.0 ** -23 * ref.abs()).all())
