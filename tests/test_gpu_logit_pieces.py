"""De-interleaving with dense logits where pieces of 1,024 froxels are dealt to XCDs: piece counts around
multiples of eight, several grids within a piece, and more pieces than workgroups; value for value a
torch gather through the site table."""
import numpy as np
import pytest
import torch

import paper_2509_24677_amd as npvs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("d,dims", [
    (4, [(8, 8, 16)]),                                          # one piece
    (4, [(8, 8, 8)] * 32), (8, [(8, 8, 8)] * 31 + [(8, 8, 16)]),  # two grids a piece
    (4, [(8, 4, 4), (40, 12, 8), (8, 4, 8)] * 10),              # pieces that end within grids
    (4, [(64, 64, 4 * k) for k in range(1, 33)]),
    (4, [(128, 64, 8), (64, 8, 8)]), (4, [(128, 64, 8), (64, 12, 8)]),  # 68 pieces, 70
    (4, [(512, 256, 64)]), (4, [(512, 256, 64), (8, 4, 4)]),    # 8,192 pieces, the last with one each; one more
    (16, [(1024, 256, 64), (32, 32, 32), (544, 16, 16)])])
def test_pieces(d, dims):
    rng = np.random.default_rng(d + len(dims))
    occ = torch.from_numpy(np.where(rng.random(sum(x * y * z for x, y, z in dims) // 8) < 4.0 / d ** 3,
                                    rng.integers(1, 256, sum(x * y * z for x, y, z in dims) // 8), 0)
                           .astype(np.uint8)).to(DEV)
    rb = npvs.build_rulebook(occ, dims, d)
    n, C = int(rb.counts[0]), d ** 3
    assert 0 < n
    Y = torch.full((rb.cap, C), float("nan"), device=DEV)
    Y[:n] = torch.randn((n, C), device=DEV, generator=torch.Generator(device=DEV).manual_seed(1))
    pvs, logits = npvs.deinterleave_threshold(Y, rb, occ, want_logits=True)
    at, key = 0, 0
    for nx, ny, nz in dims:
        bx, by, bz = nx // d, ny // d, nz // d
        row = rb.block_row[key:key + bx * by * bz].long()
        out = torch.where((row >= 0)[:, None], Y[row.clamp(min=0)], torch.full((), -float("inf"), device=DEV))
        out = out.view(bz, by, bx, d, d, d).permute(0, 3, 1, 4, 2, 5).reshape(-1)
        assert torch.equal(logits[at:at + out.numel()], out)
        bits = occ[at // 8:(at + out.numel()) // 8]
        shift = torch.arange(8, device=DEV, dtype=torch.uint8)
        want = (((out.view(-1, 8) >= 0) & (((bits[:, None] >> shift) & 1) > 0)).to(torch.uint8) << shift).sum(1)
        assert torch.equal(pvs[at // 8:(at + out.numel()) // 8], want.to(torch.uint8))
        at, key = at + out.numel(), key + bx * by * bz
    assert at == logits.numel()
