"""float32 to bfloat16 on the device, through the weight packing: round to nearest, ties to even, NaN stays a
quiet NaN with its upper bits, for every upper half of a float32 with lower halves around the ties."""
import numpy as np
import pytest
import torch

import paper_2509_24677_amd as npvs

pytestmark = pytest.mark.gpu


def test_rounding_of_packed_weights():
    low = np.array([0, 1, 0x4000, 0x7fff, 0x8000, 0x8001, 0xc000, 0xffff], np.uint32)
    u = (np.arange(1 << 16, dtype=np.uint32)[:, None] << 16 | low).reshape(-1)
    cin, cout = 160, 128
    W = np.zeros(27 * cin * cout, np.uint32)
    W[:u.size] = u
    W = W.reshape(27, cin, cout)
    got = npvs.pack_weights(torch.from_numpy(W.view(np.float32)).cuda(), npvs.NPVS_BF16).cpu().numpy()
    got = got[:2 * W.size].view(np.uint16).reshape(27, cout // 16, cin // 32, 4, 16, 8)  # [k][nb][kb][lane / 16][lane % 16][j]
    nan = (W & 0x7fffffff) > 0x7f800000
    want = np.where(nan, W >> 16 | 0x40, (W.astype(np.uint64) + 0x7fff + (W >> 16 & 1)) >> 16).astype(np.uint16)
    want = want.reshape(27, cin // 32, 4, 8, cout // 16, 16).transpose(0, 4, 1, 2, 5, 3)
    np.testing.assert_array_equal(got, want)
