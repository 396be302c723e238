"""Merging links (tpc_track_merge) of more segments than sixteen lanes each are
given for: copies of one event as frames must each have the event's links,
which the oracle confirms for the event alone elsewhere."""
import dataclasses

import numpy as np
import pytest

from tests.conftest import NB, FIT, MIN_HITS
from tpcsynth import make_config

pytestmark = pytest.mark.gpu

CHI2_RTOL = 1e-5      # the same pair by the other form: rounding of a single-precision result


@pytest.mark.parametrize("segments", [1 << 18, (1 << 18) + 1, 280_000])
def test_copies_of_an_event(segments):
    import torch
    from paper_2412_13755_amd.reco import Reco, RecoConfig
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    fr = make_config(1, scale=0.5)
    reco = Reco(RecoConfig(row_x=fr.row_x, n_sectors=fr.n_sectors, min_hits=MIN_HITS, **NB, **FIT), "cuda:0")
    dfr = reco.upload(fr)
    seeds = reco.seed(dfr, *reco.neighbours(dfr))
    tracks = reco.fit(dfr, seeds)
    T = int(seeds.n_seeds.item())
    one = [None if v is None else v[:T].clone() for v in reco.merge(seeds, tracks, 30.0)]
    assert (one[0] >= 0).sum() > 100
    copies = -(-segments // T)
    print("[merge] %d copies of %d segments, the first %d" % (copies, T, segments), flush=True)
    tile = lambda v: v[:T].repeat((copies,) + (1,) * (v.dim() - 1))[:segments].contiguous()
    at = torch.arange(copies, device="cuda:0", dtype=torch.int32).repeat_interleave(T)[:segments]
    many = dataclasses.replace(
        seeds, n_seeds=torch.full_like(seeds.n_seeds, segments), frame=at, sector=tile(seeds.sector),
        first_row=tile(seeds.first_row), offsets=torch.zeros(segments + 1, dtype=torch.int32, device="cuda:0"))
    trs = dataclasses.replace(tracks, **{k: tile(getattr(tracks, k)) for k in ("x", "par", "cov", "chi2", "ndf", "status")})
    nxt, prv, chi2, mpar, mcov, leg, lchi = reco.merge(many, trs, 30.0)
    torch.cuda.synchronize()
    whole = (segments // T) * T                            # (the last copy may lack partners)
    for got, ref in ((nxt, one[0]), (prv, one[1]), (leg, one[5])):
        want = torch.where(tile(ref) >= 0, tile(ref) + at * T, tile(ref))
        assert torch.equal(got[:whole], want[:whole])
    for got, ref in ((chi2, one[2]), (lchi, one[6])):
        a, b = got[:whole].cpu().numpy(), tile(ref)[:whole].cpu().numpy()
        np.testing.assert_allclose(a, b, rtol=CHI2_RTOL)
