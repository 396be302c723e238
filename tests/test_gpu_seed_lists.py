"""The gradient over seed lists that hold seeds the fit refuses: seeds beyond
the list's hit capacity, and a seed of a sector that does not exist.  Such
seeds contribute nothing; the workspace holds NaN beforehand."""
import dataclasses

import numpy as np
import pytest

from tests.conftest import NB, FIT, MIN_HITS
from tpcsynth import make_config

pytestmark = pytest.mark.gpu

# row sums in single precision, in another order: a few hundred terms per row
SUM_RTOL = 1e-5


@pytest.fixture(scope="module")
def event():
    import torch
    from paper_2412_13755_amd.reco import Reco, RecoConfig, DeviceFrames
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    fr = make_config(1, scale=0.05)
    reco = Reco(RecoConfig(row_x=fr.row_x, n_sectors=fr.n_sectors, min_hits=MIN_HITS, **NB, **FIT), "cuda:0")
    off = np.concatenate([fr.row_offsets, fr.row_offsets[1:] + fr.row_offsets[-1]])       # the event twice
    dfr = DeviceFrames.from_numpy(off, np.tile(fr.y, 2), np.tile(fr.z, 2), 2, fr.n_sectors, fr.n_rows, "cuda:0")
    mp = np.random.default_rng(3).normal(0, 0.05, (fr.n_sectors, fr.n_rows, 2)).astype(np.float32)
    return reco, dfr, reco.seed(dfr, *reco.neighbours(dfr)), torch.from_numpy(mp).cuda()


def _gradient(reco, dfr, seeds, mp, drop=None):
    import torch
    ws = torch.empty(reco.workspace_bytes(dfr) // 4, dtype=torch.float32, device="cuda:0").fill_(float("nan"))
    ws = ws.view(torch.uint8)
    ckpt, tracks = reco.alloc_ckpt(seeds), reco.alloc_tracks(seeds)
    tracks.status.zero_()
    reco.fit(dfr, seeds, mp, tracks=tracks, ws=ws, ckpt=ckpt)
    if drop is not None:
        tracks.status[drop] = 1
    ws.view(torch.float32).fill_(float("nan"))
    g = reco.fit_adjoint(dfr, seeds, mp, tracks, ckpt, ws=ws)
    torch.cuda.synchronize()
    return g.cpu().numpy(), tracks.status.cpu().numpy()


def test_seeds_beyond_the_hit_capacity(event):
    reco, dfr, full, mp = event
    offsets = full.to_numpy()["offsets"]
    T = len(offsets) - 1
    cap = int(offsets[T // 3]) + 2                        # in the middle of a seed
    inside = int((offsets[1:] <= cap).sum())
    part = dataclasses.replace(full, hits=full.hits[:cap], hit_yz=full.hit_yz[:cap])
    few = dataclasses.replace(part, n_seeds=full.n_seeds * 0 + inside)
    print("[lists] %d of %d seeds within capacity" % (inside, T), flush=True)
    g, status = _gradient(reco, dfr, part, mp)
    assert (status[inside:T] == 1).all() and (status[:inside] == 0).any()
    ref, _ = _gradient(reco, dfr, few, mp)
    assert np.isfinite(ref).all() and np.abs(ref).max() > 0
    assert np.array_equal(g, ref)


def test_a_seed_of_no_sector(event):
    reco, dfr, full, mp = event
    s = full.to_numpy()
    i = int((s["frame"] == 0).sum()) - 1                  # the last seed of the first frame
    ref, _ = _gradient(reco, dfr, full, mp, drop=i)
    sector = full.sector.clone()
    sector[i] = reco.cfg.n_sectors
    print("[lists] seed %d in sector %d" % (i, reco.cfg.n_sectors), flush=True)
    g, status = _gradient(reco, dfr, dataclasses.replace(full, sector=sector), mp)
    assert status[i] == 1 and np.isfinite(g).all()
    assert np.all(np.abs(g - ref) <= SUM_RTOL * np.abs(ref).max())


def test_a_map_at_any_float(event):
    import torch
    reco, dfr, full, mp = event
    ref, _ = _gradient(reco, dfr, full, mp)
    odd = torch.empty(mp.numel() + 1, device="cuda:0")[1:].view(mp.shape)
    odd.copy_(mp)
    assert odd.data_ptr() % 8 == 4
    g, _ = _gradient(reco, dfr, full, odd)
    assert np.array_equal(g, ref)


def test_a_fitted_segment_of_no_sector(event):
    # the first seed in a sector below the first: its legs are not looked for
    # there, and the others' are theirs
    import torch
    reco, dfr, full, _ = event
    T = int(full.n_seeds.item())
    tracks = reco.fit(dfr, full)
    assert int(tracks.status[0].item()) == 0
    sector = full.sector.clone()
    sector[0] = -1
    leg, lchi = reco.merge(dataclasses.replace(full, sector=sector), tracks, 30.0)[5:7]
    tracks.status[0] = 1
    ref, rchi = reco.merge(full, tracks, 30.0)[5:7]
    assert (ref[:T] >= 0).any()
    assert torch.equal(leg[1:T], ref[1:T]) and torch.equal(lchi[1:T], rchi[1:T])
    assert int(leg[0].item()) == -1
