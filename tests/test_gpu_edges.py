"""The sizes at which a kernel or its launch changes form, each against the
oracle (integers and bytes equal) or, for the adjoint, against the gradient
of another checkpoint interval.

 - the rANS coder's three coding loops: small L, a symbol of more than half
   the frequency table, frequencies of one, tables in and out of LDS, and
   block counts around those of the two workgroup sizes;
 - seeding where the placement sums the segments' counts itself and where it
   reads scanned counts, and with several wavefronts per segment;
 - the skip search with one query's windows beyond the pool of candidates,
   pools of several batches, rows around one pass of queries, and ties;
 - track following over rows around the size that is indexed in LDS, and
   with as many seeds as take 8, 16, 32 and 64 lanes of a wavefront;
 - the adjoint's checkpoint intervals below, at and above its tape of four
   rows, and intervals that do not divide by it.
"""
import numpy as np
import pytest

import oracle
from tests.conftest import NB, FIT, MIN_HITS
from tests import parity
from tests.test_gpu_adjoint import GRAD_RTOL
from tests.test_gpu_follow import compare_follow, GATE, MAX_MISS
from tests.test_gpu_rans import _check as check_stream
from tpcsynth import make_config

pytestmark = pytest.mark.gpu


def _upload(off, y, z, n_frames, n_rows, **cfg):
    import torch
    from paper_2412_13755_amd.reco import Reco, RecoConfig, DeviceFrames
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    row_x = np.linspace(85.0, 85.0 + n_rows - 1, n_rows).astype(np.float32)
    reco = Reco(RecoConfig(row_x=row_x, n_sectors=1, min_hits=MIN_HITS, **{**NB, **cfg}, **FIT), "cuda:0")
    return reco, DeviceFrames.from_numpy(off, y, z, n_frames, 1, n_rows, "cuda:0"), row_x


def _lines(tracks, n_rows, seed, width=0.0):
    """Straight tracks through every row, one sector per frame: row offsets, y
    and z.  tracks: the tracks of each frame; width: their extent in y and z
    (default: about one track per search window)."""
    rng = np.random.default_rng(seed)
    off, ys, zs = [0], [], []
    for n in tracks:
        w = width or 3.0 * np.sqrt(max(n, 1))
        a, c = rng.uniform(-w / 2, w / 2, n), rng.uniform(0, w, n)
        b, d = rng.uniform(-0.2, 0.2, n), rng.uniform(-0.2, 0.2, n)
        for r in range(n_rows):
            keep = rng.random(n) < 0.97
            ys.append((a + b * r + rng.normal(0, 0.03, n))[keep])
            zs.append((c + d * r + rng.normal(0, 0.03, n))[keep])
            off.append(off[-1] + int(keep.sum()))
    cat = lambda v: np.concatenate(v).astype(np.float32)
    return np.array(off, np.int32), cat(ys), cat(zs)


def _symbols(kind, n):
    rng = np.random.default_rng(n % 1009 + len(kind))
    if kind == "one_of_two_rare":             # f > M / 2 and f = 1
        x = np.zeros(n, np.int64)
        x[:: max(1, n // 3)] = 1
    elif kind == "four":
        x = rng.integers(0, 4, n)
    elif kind == "one":
        x = np.full(n, 12345)
    elif kind == "two_even":
        x = rng.integers(0, 2, n)
    elif kind == "rare":                      # most of the symbols with f = 1
        x = np.where(rng.random(n) < 0.9, rng.integers(0, 8, n), rng.integers(0, 200, n))
    else:                                     # "wide": the table stays in global memory
        x = rng.integers(0, 12000, n)
    return x.astype(np.int32)


@pytest.mark.parametrize("kind,L,B,n", [
    ("two_even", 1, 64, 1000), ("four", 2, 64, 4096), ("four", 7, 128, 5001), ("four", 8, 128, 5001),
    ("two_even", 9, 64, 777), ("one_of_two_rare", 12, 256, 20_001), ("one_of_two_rare", 16, 1024, 20_001),
    ("one", 8, 64, 1), ("one", 16, 128, 4097), ("rare", 8, 64, 30_011), ("rare", 12, 4096, 30_011),
    ("wide", 14, 8192, 200_003), ("rare", 10, 64, 64 * 5119), ("rare", 10, 64, 64 * 5119 + 1),
    ("one_of_two_rare", 10, 64, 64 * 5200 + 17), ("rare", 12, 256, 256 * 5121 + 5), ("wide", 14, 64, 64 * 5200 + 17)])
def test_coding_loops(kind, L, B, n):
    check_stream(_symbols(kind, n), L, B, kind)


@pytest.mark.parametrize("frames,n_rows,tracks", [
    (512, 16, 3), (513, 16, 3), (127, 129, 2), (1024, 16, 2), (1, 16, 511), (1, 16, 560), (3, 16, 900)])
def test_seeding_sizes(frames, n_rows, tracks):
    import torch
    n = np.random.default_rng(frames).integers(0, 2 * tracks, frames) if tracks < 100 else [tracks] * frames
    off, y, z = _lines(n, n_rows, frames + tracks)
    print("[edges] seeding: %d frames of %d rows, N=%d" % (frames, n_rows, off[-1]), flush=True)
    reco, dfr, _ = _upload(off, y, z, frames, n_rows)
    up, dn = reco.neighbours(dfr)
    seeds = reco.seed(dfr, up, dn)
    torch.cuda.synchronize()
    ru, rd = oracle.neighbours(off, y, z, n_rows, **NB)
    np.testing.assert_array_equal(up.cpu().numpy(), ru)
    np.testing.assert_array_equal(dn.cpu().numpy(), rd)
    sd = oracle.ca_seed(off, ru, rd, 1, n_rows, MIN_HITS)
    assert int(seeds.status.item()) == 0 and len(sd["frame"]) > 0
    parity.assert_seeds_equal(seeds.to_numpy(), sd)


# clusters per row (five rows), extent in cm, coordinates rounded to this
SKIP = {
    "one_each": ((1, 1, 1, 1, 1), 0.4, 0.0),
    "a_pass_of_queries": ((50, 60, 256, 60, 50), 20.0, 0.0),
    "a_query_more": ((50, 60, 257, 60, 50), 20.0, 0.0),
    "three_passes": ((90, 100, 700, 100, 90), 30.0, 0.0),
    "several_batches": ((300, 300, 256, 300, 300), 10.0, 0.0),
    "pool_just_full": ((512, 512, 9, 512, 512), 1.0, 0.0),
    "beyond_the_pool": ((512, 512, 9, 513, 512), 1.0, 0.0),
    "far_beyond_the_pool": ((1000, 1010, 20, 1020, 1024), 1.0, 0.0),
    "a_dense_partner": ((20, 60, 40, 1025, 30), 20.0, 0.0),
    "ties": ((150, 150, 300, 150, 150), 10.0, 0.5),
    "ties_beyond_the_pool": ((600, 600, 30, 600, 600), 1.0, 0.25),
}


@pytest.mark.parametrize("name", sorted(SKIP))
def test_skip_stacks(name):
    import torch
    rows, ext, grid = SKIP[name]
    rng = np.random.default_rng(7)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    y, z = rng.uniform(-ext / 2, ext / 2, off[-1]), rng.uniform(10, 10 + ext, off[-1])
    if grid:
        y, z = np.round(y / grid) * grid, np.round(z / grid) * grid
    y, z = y.astype(np.float32), z.astype(np.float32)
    if off[-1] > 50:
        y[3], z[off[3] - 2], y[off[-1] - 2] = np.nan, np.inf, -np.inf
    print("[edges] skip %s: N=%d" % (name, off[-1]), flush=True)
    reco, dfr, _ = _upload(off, y, z, 1, 5)
    up, dn = reco.neighbours_skip(dfr)
    torch.cuda.synchronize()
    ru, rd = oracle.neighbours_skip(off, y, z, 5, **NB)
    np.testing.assert_array_equal(up.cpu().numpy(), ru)
    np.testing.assert_array_equal(dn.cpu().numpy(), rd)


@pytest.mark.parametrize("frames,tracks", [(1, 2040), (1, 2300), (4, 1200), (9, 1500), (15, 1500)])
def test_following_sizes(frames, tracks):
    import torch
    n_rows = 12
    off, y, z = _lines([tracks] * frames, n_rows, tracks)
    longest = int(np.diff(off).max())
    assert (longest <= 2048) == (tracks < 2300)
    reco, dfr, row_x = _upload(off, y, z, frames, n_rows)
    up, dn = reco.neighbours(dfr)
    seeds = reco.seed(dfr, up, dn)
    rows, tr = reco.follow(dfr, seeds, GATE, MAX_MISS)
    torch.cuda.synchronize()
    ru, rd = oracle.neighbours(off, y, z, n_rows, **NB)
    sd = oracle.ca_seed(off, ru, rd, 1, n_rows, MIN_HITS)
    parity.assert_seeds_equal(seeds.to_numpy(), sd)
    r = oracle.follow(sd, off, y, z, row_x, 1, n_rows, gate=GATE, max_miss=MAX_MISS, **FIT)
    T = len(sd["frame"])
    print("[edges] follow: %d seeds, rows of up to %d clusters" % (T, longest), flush=True)
    g = {k: getattr(tr, k)[:T].cpu().numpy() for k in ("x", "par", "cov", "chi2", "ndf", "status")}
    g["rows"] = rows[:T].cpu().numpy()
    print("[edges] follow:", compare_follow(g, r), flush=True)
    # the first rows order the work and decide nothing
    seeds.first_row.random_(-2**31, 2**31 - 1)
    rows2, tr2 = reco.follow(dfr, seeds, GATE, MAX_MISS)
    assert torch.equal(rows2[:T], rows[:T]) and torch.equal(tr2.status[:T], tr.status[:T])
    assert np.array_equal(tr2.par[:T].cpu().numpy(), g["par"], equal_nan=True)


def test_adjoint_checkpoint_intervals():
    import torch
    from paper_2412_13755_amd.reco import Reco, RecoConfig, KalmanChi2
    fr = make_config(4, scale=0.01)
    mp = np.random.default_rng(1).normal(0, 0.05, (fr.n_sectors, fr.n_rows, 2)).astype(np.float32)
    grads = {}
    for k in (16, 1, 2, 3, 4, 5, 7, 64):
        print("[edges] checkpoints every %d rows" % k, flush=True)
        reco = Reco(RecoConfig(row_x=fr.row_x, n_sectors=fr.n_sectors, min_hits=MIN_HITS, ckpt_rows=k, **NB,
                               **FIT), "cuda:0")
        dfr = reco.upload(fr)
        seeds = reco.seed(dfr, *reco.neighbours(dfr))
        m = torch.from_numpy(mp).cuda().requires_grad_(True)
        KalmanChi2.apply(m, reco, dfr, seeds).backward()
        torch.cuda.synchronize()
        grads[k] = m.grad.cpu().numpy().astype(np.float64)
    ref = grads[16]
    floor = 1e-3 * np.abs(ref).max()
    assert floor > 0
    for k, g in grads.items():
        assert np.linalg.norm(g - ref) <= GRAD_RTOL * np.linalg.norm(ref), k
        assert np.all(np.abs(g - ref) <= GRAD_RTOL * np.maximum(np.abs(ref), floor)), k
