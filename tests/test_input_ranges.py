"""The input ranges of the general BF16 kernel (1024 or more inputs, given a workspace): none is empty,
since a workgroup of an empty range has no stage to load.  The number of ranges is read from the
workspace size: one float32 partial result [cap][cout] each."""
import ctypes

import pytest
import torch

import paper_2509_24677_amd as npvs
from paper_2509_24677_amd import _lib as L

DEV = "cuda"


def ranges(cin):
    n = ctypes.c_size_t()
    L.call("npvs_conv_fwd_workspace_size", cin, 8, 1, L.NPVS_BF16, ctypes.byref(n))
    assert n.value % (4 * 8) == 0
    return max(1, n.value // (4 * 8))


def test_no_range_is_empty():
    for chunks in range(1, 1025):  # of 32 inputs
        for cin in (32 * chunks - 24, 32 * chunks):
            kz = ranges(cin)
            per = -(-chunks // kz)  # chunks of every range but the last, as the kernel divides them
            assert (kz - 1) * per < chunks, (cin, kz, per)
            assert kz == 1 if chunks < 32 else 1 < kz <= 16


@pytest.mark.gpu
@pytest.mark.parametrize("sites", [1, 17, 400])
@pytest.mark.parametrize("cin", [2592, 2848, 4128])  # 81, 89 and 129 chunks, in ranges of nine
@pytest.mark.parametrize("cout", [8, 72])
def test_ragged_ranges(sites, cin, cout):
    from test_gpu_f32_matrix import rows, rulebook

    rb, _ = rulebook(sites, sites)
    gen = torch.Generator(device=DEV).manual_seed(cin + cout)
    X = rows(sites, cin, rb.cap, gen).to(torch.bfloat16)  # rows past the sites NaN: never read
    W = torch.randn((27, cin, cout), generator=gen, device=DEV)
    Wp = npvs.pack_weights(W, npvs.NPVS_BF16)
    got, want = (npvs.sparse_conv_fwd(X, Wp, None, cin, cout, rb, npvs.NPVS_BF16, False, out_f32=True, variant=v)
                 for v in (None, 5))
    assert torch.equal(got[:sites], want[:sites])
    pick = torch.tensor(sorted({0, sites // 2, sites - 1}), device=DEV)
    ref = torch.zeros((len(pick), cout), dtype=torch.float64, device=DEV)
    mag = torch.zeros_like(ref)
    Wd = W.to(torch.bfloat16).double()
    for k in range(27):
        i = rb.nbr[k, pick].long()
        x = torch.where((i >= 0)[:, None], X[i.clamp(min=0)].double(), torch.zeros((), dtype=torch.float64, device=DEV))
        ref += x @ Wd[k]
        mag += x.abs() @ Wd[k].abs()
    # float32 accumulation of 27 cin products: half an ulp of the running sum each, at most
    assert bool(((got[pick].double() - ref).abs() <= 27 * cin * 2.0 ** -24 * mag + 2.0 ** -23 * ref.abs()).all())
