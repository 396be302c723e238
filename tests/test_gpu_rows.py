"""Links of single row triplets (tpc_neighbours) against the oracle,
bit-exact, at the sizes where the search of a row changes its form: the two
neighbouring rows together at and above the small LDS form's 1152 clusters,
either row at and above the large form's 1024, h-rows of more than one
workgroup's 256 clusters, windows around the list lengths of 16 and 24
clusters, windows of everything (taken by a wavefront, beyond its lists in
four parts), ties on a coarse grid, and non-finite clusters.  Each triplet is
searched alone (one workgroup per segment) and among empty frames (frames of
small rows: the large rows are looked for).
"""
import numpy as np
import pytest

import oracle
from tests.conftest import NB, FIT, MIN_HITS

pytestmark = pytest.mark.gpu

# (down, h, up clusters), extent in y and z in cm, coordinates rounded to this
CASES = {
    "one_each": ((1, 1, 1), 0.4, 0.4, 0.0),
    "no_down": ((0, 40, 40), 5.0, 5.0, 0.0),
    "no_up": ((40, 40, 0), 5.0, 5.0, 0.0),
    "small_form_full": ((576, 300, 576), 40.0, 200.0, 0.0),
    "small_form_uneven": ((1024, 257, 128), 40.0, 200.0, 0.0),
    "large_form_first": ((577, 300, 576), 40.0, 200.0, 0.0),
    "large_form_full": ((1024, 700, 1024), 40.0, 200.0, 0.0),
    "dense": ((1025, 100, 64), 40.0, 200.0, 0.0),
    "long_h_row": ((30, 2000, 30), 30.0, 60.0, 0.0),
    "windows_of_16": ((120, 200, 120), 16.0, 24.0, 0.0),
    "windows_of_24": ((600, 200, 600), 36.0, 64.0, 0.0),
    "window_of_1000": ((500, 65, 500), 1.0, 1.0, 0.0),
    "window_beyond_small_lists": ((560, 40, 592), 1.0, 1.0, 0.0),
    "window_beyond_large_lists": ((1000, 40, 1010), 1.0, 1.0, 0.0),
    "ties": ((300, 300, 300), 20.0, 40.0, 0.5),
    "ties_in_one_window": ((600, 70, 600), 2.0, 2.0, 0.25),
}


def _triplet(name, seed):
    (n0, n, n1), ey, ez, grid = CASES[name]
    rng = np.random.default_rng(seed)
    m = n0 + n + n1
    y = rng.uniform(-ey / 2, ey / 2, m)
    z = rng.uniform(10.0, 10.0 + ez, m)
    if grid:
        y, z = np.round(y / grid) * grid, np.round(z / grid) * grid
    y, z = y.astype(np.float32), z.astype(np.float32)
    if m > 50:                                   # (one of each kind per row, where there is one)
        for k, v in ((3, np.nan), (m // 2, np.inf), (m - 2, -np.inf)):
            y[k] = v
            z[k + 1] = -v
    return np.array([0, n0, n0 + n, m], np.int32), y, z


@pytest.mark.parametrize("empty", [0, 3000])
@pytest.mark.parametrize("name", sorted(CASES))
def test_row_triplet(name, empty):
    import torch
    from paper_2412_13755_amd.reco import Reco, RecoConfig, DeviceFrames
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    print("[rows] %s, %d empty frames" % (name, empty), flush=True)
    off, y, z = _triplet(name, 5)
    ru, rd = oracle.neighbours(off, y, z, 3, **NB)
    ends = np.concatenate([off, np.full(3 * empty, off[-1], np.int32)]).astype(np.int32)
    cfg = RecoConfig(row_x=np.array([85.0, 86.0, 87.0], np.float32), n_sectors=1, min_hits=MIN_HITS, **NB, **FIT)
    reco = Reco(cfg, "cuda:0")
    dfr = DeviceFrames.from_numpy(ends, y, z, 1 + empty, 1, 3, "cuda:0")
    up, dn = reco.neighbours(dfr)
    pup, pdn, _, _ = reco.reconstruct(dfr, "persistent")
    for form, u, d in (("staged", up, dn), ("persistent", pup, pdn)):
        assert np.array_equal(u.cpu().numpy(), ru), form
        assert np.array_equal(d.cpu().numpy(), rd), form
