"""Links of single row triplets in windows that hold most of a row
(tpc_neighbours) against the oracle, bit-exact: where a wavefront takes a
cluster's pairs one by one and where it searches boxes around predictions
(more than 1024 pairs in cells made for that), for rows of the small and the
large LDS form; windows and cuts of one axis only, cuts of more than the
window, of nothing and without limit, ties, and non-finite clusters.  Each
triplet is searched staged and by the persistent kernel."""
import numpy as np
import pytest

import oracle
from tests.conftest import NB, FIT, MIN_HITS

pytestmark = pytest.mark.gpu

INF = float("inf")
# (down, h, up clusters), extents in y and z, (win_y, win_z, cut_y, cut_z), coordinates rounded to this
CASES = {
    "pairs_1024": ((32, 100, 32), 20.0, 100.0, (40.0, 200.0, 0.6, 0.75), 0.0),
    "pairs_1056": ((33, 100, 32), 20.0, 100.0, (40.0, 200.0, 0.6, 0.75), 0.0),
    "one_up": ((700, 40, 1), 20.0, 100.0, (40.0, 200.0, 0.6, 0.75), 0.0),
    "one_down": ((1, 40, 700), 20.0, 100.0, (40.0, 200.0, 20.0, 20.0), 0.0),
    "ups_64": ((200, 70, 64), 20.0, 100.0, (40.0, 200.0, 0.6, 0.75), 0.0),
    "ups_65": ((200, 70, 65), 20.0, 100.0, (40.0, 200.0, 0.6, 0.75), 0.0),
    "event": ((230, 300, 230), 36.0, 250.0, (40.0, 40.0, 0.6, 0.75), 0.0),
    "small_form_full": ((576, 130, 576), 40.0, 250.0, (80.0, 300.0, 0.6, 0.75), 0.0),
    "large_form_full": ((1024, 130, 1024), 40.0, 250.0, (80.0, 300.0, 0.6, 0.75), 0.0),
    "narrow_in_y": ((400, 100, 400), 36.0, 250.0, (1.0, 200.0, 0.6, 0.75), 0.0),
    "narrow_in_z": ((400, 100, 400), 36.0, 250.0, (40.0, 5.0, 0.6, 0.75), 0.0),
    "cut_of_one_axis": ((300, 100, 300), 36.0, 250.0, (10.0, 100.0, 20.0, 0.75), 0.0),
    "cuts_of_the_window": ((600, 60, 500), 36.0, 250.0, (20.0, 100.0, 20.0, 100.0), 0.0),
    "no_cuts": ((560, 20, 560), 36.0, 250.0, (20.0, 100.0, INF, INF), 0.0),
    "no_cuts_beyond_the_lists": ((1000, 20, 1000), 36.0, 250.0, (80.0, 300.0, INF, INF), 0.0),
    "cuts_of_almost_nothing": ((500, 200, 500), 36.0, 250.0, (80.0, 300.0, 0.1, 0.1), 0.0),
    "a_window_of_everything": ((500, 100, 500), 36.0, 250.0, (1e30, 1e30, 0.6, 0.75), 0.0),
    "ties": ((300, 200, 300), 20.0, 40.0, (30.0, 50.0, 1.1, 1.1), 0.5),
    "ties_large_form": ((900, 100, 900), 10.0, 20.0, (30.0, 50.0, 1.1, 1.1), 0.5),
    "all_of_one_y": ((400, 100, 400), 0.0, 250.0, (40.0, 200.0, 0.6, 0.75), 0.0),
}


def _triplet(name):
    (n0, n, n1), ey, ez, _, grid = CASES[name]
    rng = np.random.default_rng(len(name))
    m = n0 + n + n1
    y, z = rng.uniform(-ey / 2, ey / 2, m), rng.uniform(0.0, ez, m)
    if grid:
        y, z = np.round(y / grid) * grid, np.round(z / grid) * grid
    return np.array([0, n0, n0 + n, m], np.int32), y.astype(np.float32), z.astype(np.float32)


@pytest.mark.parametrize("infinite", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_wide_windows(name, infinite):
    import torch
    from paper_2412_13755_amd.reco import Reco, RecoConfig, DeviceFrames
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    off, y, z = _triplet(name)
    nb = dict(zip(("win_y", "win_z", "cut_y", "cut_z"), CASES[name][3]))
    assert set(nb) == set(NB)
    if infinite:
        if min(np.diff(off)) < 10:
            pytest.skip("rows too short to lose clusters")
        y[3], z[off[1] + 4], y[off[2] + 1], z[off[2] + 5] = np.nan, np.inf, -np.inf, np.nan
    ru, rd = oracle.neighbours(off, y, z, 3, **nb)
    print("[wide] %s: %d of %d link" % (name, (ru >= 0).sum(), off[2] - off[1]), flush=True)
    assert (ru >= 0).any() or name in ("one_up", "one_down")
    cfg = RecoConfig(row_x=np.array([85.0, 86.0, 87.0], np.float32), n_sectors=1, min_hits=MIN_HITS, **nb, **FIT)
    reco = Reco(cfg, "cuda:0")
    dfr = DeviceFrames.from_numpy(off, y, z, 1, 1, 3, "cuda:0")
    up, dn = reco.neighbours(dfr)
    pup, pdn, _, _ = reco.reconstruct(dfr, "persistent")
    for form, u, d in (("staged", up, dn), ("persistent", pup, pdn)):
        assert np.array_equal(u.cpu().numpy(), ru), form
        assert np.array_equal(d.cpu().numpy(), rd), form
