"""The skip search (tpc_neighbours_skip) around its pool of 2048 window
candidates, against the oracle, bit-exact: the clusters of row 2 have no
adjacent partners above (row 3 is empty), so they are queried, and the rows
around them hold exactly as many candidates as a case is named for: a query
that fills the pool, one beyond it (taken by its thread alone), far beyond
it, two queries of half a pool each, many small ones in several batches,
ties, and a dense partner row.  The counts are asserted from the data."""
import numpy as np
import pytest

import oracle
from tests.conftest import NB, FIT, MIN_HITS

pytestmark = pytest.mark.gpu

POOL, ROW_MAX = 2048, 1024

# clusters of rows 0, 1, 2, 4; extent in cm; coordinates rounded to this
CASES = {
    "pool_just_full": ((513, 512, 9, 1023), 1.0, 0.0),
    "one_beyond_the_pool": ((514, 512, 9, 1023), 1.0, 0.0),
    "one_less_than_the_pool": ((512, 512, 9, 1023), 1.0, 0.0),
    "far_beyond_the_pool": ((1000, 1010, 20, 1024), 1.0, 0.0),
    "two_halves": ((256, 256, 30, 512), 1.0, 0.0),
    "two_halves_and_one": ((257, 256, 30, 512), 1.0, 0.0),
    "several_batches": ((600, 600, 300, 900), 10.0, 0.0),
    "batches_with_some_beyond": ((700, 1000, 300, 700), 4.5, 0.0),
    "ties": ((500, 500, 100, 500), 4.0, 0.5),
    "ties_beyond_the_pool": ((900, 900, 30, 1000), 1.0, 0.25),
    "dense_partner": ((600, 600, 100, 1100), 2.0, 0.0),
}
# clusters that a query's windows hold: least and most over the queries
EXPECT = {
    "pool_just_full": (POOL, POOL),
    "one_beyond_the_pool": (POOL + 1, POOL + 1),
    "one_less_than_the_pool": (POOL - 1, POOL - 1),
    "far_beyond_the_pool": (POOL + 900, 3100),
    "two_halves": (POOL // 2, POOL // 2),
    "two_halves_and_one": (POOL // 2 + 1, POOL // 2 + 1),
    "several_batches": (50, POOL - 1),
    "batches_with_some_beyond": (500, 2400),
    "ties": (500, POOL - 1),
    "ties_beyond_the_pool": (POOL + 1, 2800),
    "dense_partner": (0, 2300),
}


def _frame(name):
    (n0, n1, n2, n4), ext, grid = CASES[name]
    rows = (n0, n1, n2, 0, n4)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    rng = np.random.default_rng(11)
    y, z = rng.uniform(-ext / 2, ext / 2, off[-1]), rng.uniform(10.0, 10.0 + ext, off[-1])
    if grid:
        y, z = np.round(y / grid) * grid, np.round(z / grid) * grid
    return off, y.astype(np.float32), z.astype(np.float32)


def _candidates(off, y, z):
    """Per cluster of row 2: clusters of rows 0, 1, 3, 4 in its windows."""
    f = np.float32
    out = []
    for h in range(off[2], off[3]):
        n = 0
        for r, d in ((0, 2), (1, 1), (3, 1), (4, 2)):
            s = slice(off[r], off[r + 1])
            n += int(((np.abs(y[s] - y[h]) <= f(d) * f(NB["win_y"])) & (np.abs(z[s] - z[h]) <= f(d) * f(NB["win_z"]))).sum())
        out.append(n)
    return np.array(out)


@pytest.mark.parametrize("infinite", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_pool(name, infinite):
    import torch
    from paper_2412_13755_amd.reco import Reco, RecoConfig, DeviceFrames
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    off, y, z = _frame(name)
    lo, hi = EXPECT[name]
    c = _candidates(off, y, z)
    if lo > 0:
        assert lo <= c.min() and c.max() <= hi, (c.min(), c.max())
    if name == "several_batches":
        assert c.sum() > 4 * POOL
    if name == "batches_with_some_beyond":
        assert (c > POOL).any() and (c <= POOL).any()
    assert (max(np.diff(off)) > ROW_MAX) == (name == "dense_partner")
    if infinite:                                  # a query and a candidate of every row fewer
        for k, v in ((off[0] + 1, np.nan), (off[1] + 2, np.inf), (off[2] + 1, -np.inf), (off[4] + 3, np.nan)):
            y[k] = v
        z[off[4] + 5] = np.inf
    ru, _ = oracle.neighbours(off, y, z, 5, **NB)
    su, sd = oracle.neighbours_skip(off, y, z, 5, **NB)
    row2 = slice(off[2], off[3])
    assert (ru[row2] < 0).all() and (su[row2] >= 0).sum() > 3
    print("[pool] %s: N=%d, %d to %d candidates, %d of %d queries link" % (
        name, off[-1], c.min(), c.max(), (su[row2] >= 0).sum(), off[3] - off[2]), flush=True)
    cfg = RecoConfig(row_x=np.linspace(85.0, 89.0, 5).astype(np.float32), n_sectors=1, min_hits=MIN_HITS, **NB, **FIT)
    reco = Reco(cfg, "cuda:0")
    dfr = DeviceFrames.from_numpy(off, y, z, 1, 1, 5, "cuda:0")
    up, dn = reco.neighbours_skip(dfr)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(up.cpu().numpy(), su)
    np.testing.assert_array_equal(dn.cpu().numpy(), sd)
