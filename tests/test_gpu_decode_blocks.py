"""rANS streams (tpc_rans_encode, tpc_rans_decode) of the numbers of blocks
where the decoder deals them out differently, with the slot table in LDS
(L = 8, 14) and in global memory (L = 16): the oracle's bytes, and the symbols
back."""
import numpy as np
import pytest

from tests.test_gpu_rans import _check as check_stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [8, 14, 16])
@pytest.mark.parametrize("blocks", [1, 15, 16, 17, 255, 2047, 2048, 2049])
def test_blocks(blocks, L):
    rng = np.random.default_rng(blocks + L)
    n = 64 * blocks - (13 if blocks % 2 else 0)
    x = rng.normal(0, 9.0, n).round().astype(np.int32)
    check_stream(x, L, 64, "%d blocks" % blocks)
    import torch
    from paper_2412_13755_amd.reco import rans_encode, rans_decode
    out, size, status = rans_encode(torch.from_numpy(x).cuda(), L, 64)
    assert int(status.item()) == 0
    k = int(size.item())
    y, count, status = rans_decode(out[:k].clone(), k, n)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and int(count.item()) == n
    assert np.array_equal(y[:n].cpu().numpy(), x)
    # a word more than the blocks use is found out
    words = torch.zeros(k // 4 + 2, dtype=torch.int32, device="cuda:0")
    bad = words.view(torch.uint8)
    bad[:k] = out[:k]
    words[10 + (int(words[9].item()) + 3) // 4 + blocks] += 1       # the last block's end
    _, _, status = rans_decode(bad, k + 2, n)
    assert int(status.item()) == -1
