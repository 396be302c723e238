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
    check_stream(rng.normal(0, 9.0, n).round().astype(np.int32), L, 64, "%d blocks" % blocks)
