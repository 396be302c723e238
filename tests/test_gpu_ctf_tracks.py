"""The residual transform (tpc_ctf_build) of made-up tracks against the oracle,
array by array, at the numbers of tracks where its counts and prefixes
change form: around one workgroup's prefixes (1024 tracks) and around the
number beyond which tracks that are not kept are not read (65536)."""
import numpy as np
import pytest

import oracle
from tests.conftest import NB, FIT, MIN_HITS

pytestmark = pytest.mark.gpu

ROWS, Q = 12, 0.01


@pytest.mark.parametrize("kept", [0.0, 0.4, 1.0])
@pytest.mark.parametrize("T", [0, 1, 64, 1023, 1024, 1025, 5000, 65535, 65536, 65537, 70001])
def test_tracks(T, kept):
    import torch
    from paper_2412_13755_amd.reco import Reco, RecoConfig, DeviceFrames
    from paper_2412_13755_amd import _capi as C
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    rng = np.random.default_rng(T)
    n = max(T // 2, 3)                                    # clusters per row: each in about two tracks
    off = (np.arange(ROWS + 1) * n).astype(np.int32)
    y, z = (rng.normal(0, s, off[-1]).astype(np.float32) for s in (10.0, 100.0))
    rows = rng.integers(0, n, (T, ROWS)) + off[:ROWS]
    rows = np.where(rng.random((T, ROWS)) < 0.7, rows, -1).astype(np.int32)
    status = np.where(rng.random(T) < kept, 0, rng.integers(1, 5, T)).astype(np.int32)
    zero = np.zeros(T, np.int32)
    row_x = np.linspace(85.0, 96.0, ROWS).astype(np.float32)
    reco = Reco(RecoConfig(row_x=row_x, n_sectors=1, min_hits=MIN_HITS, **NB, **FIT), "cuda:0")
    dfr = DeviceFrames.from_numpy(off, y, z, 1, 1, ROWS, "cuda:0")
    seeds = reco.alloc_seeds(dfr, cap_seeds=T + 7)
    seeds.n_seeds.fill_(T)
    seeds.frame.zero_()
    seeds.sector.zero_()
    tr = reco.alloc_tracks(seeds)
    drows = torch.full((T + 7, ROWS), 1, dtype=torch.int32, device="cuda:0")
    tr.status.zero_()
    drows[:T], tr.status[:T] = torch.from_numpy(rows).cuda(), torch.from_numpy(status).cuda()
    ws = torch.full((64 * (T + 7) + 64 * int(off[-1]) + (1 << 20),), 0x55, dtype=torch.uint8, device="cuda:0")
    print("[ctf] %d tracks, %d kept" % (T, (status == 0).sum()), flush=True)
    out = reco.ctf_build(dfr, seeds, drows, tr, Q, Q, ws=ws)
    torch.cuda.synchronize()
    ref = oracle.ctf_build(off, y, z, 1, ROWS, rows, status, zero, zero, Q, Q)
    counts = out["counts"].cpu().numpy()
    for i, k in enumerate(C.CTF_ARRAYS):
        assert counts[i] == len(ref[k]), k
        np.testing.assert_array_equal(out[k][:counts[i]].cpu().numpy(), ref[k], err_msg=k)
