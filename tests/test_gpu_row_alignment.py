"""Rows at an address that is not 16-byte aligned (a slice of a buffer) give the rows' own result bit for
bit, through every shape the BF16 dispatch has for them and through the FP32 kernel."""
import pytest
import torch

import paper_2509_24677_amd as npvs
from test_gpu_f32_matrix import rows, rulebook

pytestmark = pytest.mark.gpu
DEV = "cuda"


def shifted(X, by):
    buf = torch.full((X.numel() + by,), float("nan"), dtype=X.dtype, device=DEV)
    t = buf[by:].view(X.shape)
    t.copy_(X)
    assert t.data_ptr() % 16 == by * X.element_size()
    return t


@pytest.mark.parametrize("sites", [1, 300, 20000])
@pytest.mark.parametrize("cin,cout", [(8, 8), (8, 64), (40, 64), (64, 64), (64, 72), (96, 64)])
def test_bf16_rows(sites, cin, cout):
    rb, _ = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin * 100 + cout)
    X = rows(sites, cin, rb.cap, gen).to(torch.bfloat16)
    Wp = npvs.pack_weights(torch.randn((27, cin, cout), generator=gen, device=DEV), npvs.NPVS_BF16)
    fwd = lambda x: npvs.sparse_conv_fwd(x, Wp, None, cin, cout, rb, npvs.NPVS_BF16, False, out_f32=True)[:sites]
    want = fwd(X)
    assert bool(torch.isfinite(want).all())
    for by in (1, 2, 4):
        assert torch.equal(fwd(shifted(X, by)), want), by


@pytest.mark.parametrize("sites", [1, 300, 9000])
@pytest.mark.parametrize("cin,cout", [(16, 64), (64, 33), (256, 64), (260, 64), (512, 16), (512, 20)])
def test_f32_rows(sites, cin, cout):
    rb, _ = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin * 100 + cout)
    X = rows(sites, cin, rb.cap, gen)
    Wp = npvs.pack_weights(torch.randn((27, cin, cout), generator=gen, device=DEV), npvs.NPVS_F32)
    fwd = lambda x: npvs.sparse_conv_fwd(x, Wp, None, cin, cout, rb, npvs.NPVS_F32, False)[:sites]
    want = fwd(X)
    assert bool(torch.isfinite(want).all())
    for by in (1, 2, 3):
        assert torch.equal(fwd(shifted(X, by)), want), by
