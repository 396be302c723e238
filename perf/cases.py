"""The work that programs give this library, as measurable cases.

Each case is one pass through the public entry points of
``paper_2412_13755_amd.reco`` on synthetic time frames: helices from the
origin through 152 pad-row planes, smeared, with noise clusters, loopers and
truncated tracks (the sizes are those of the repository's workloads and
benchmark legs: a 200-track sector, a 10^4-track event, a continuous-readout
frame, 64 uneven frames, 10^5 tracks with a distortion map, arrays of 2^28
symbols).  The frames are made on the GPU from the seed alone.

``exact`` computes what a pass returns with plain torch in 64 bits (searches
and comparisons in single precision, which defines the links exactly).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2412_13755_amd import reco as R

DEV = "cuda:0"
ROWS = 152
C_LIGHT = 0.00299792458
TAN10 = math.tan(math.radians(10.0))
DRIFT, R_OUTER, V_DRIFT = 250.0, 250.0, 2.5
GATE, MAX_MISS = 25.0, 3                      # track following
MERGE_CUT = 30.0
X0, PION, CUT = 2870.0, 0.13957, 30.0         # gas: radiation length, mass hypothesis, rejection
GAS = (0.948e-3, 0.4966, 121.8e-9)            # Ne-CO2-N2: density, Z/A, mean excitation energy
CTF_Q = 0.01                                  # quantisation of y and z (cm)
RANS_L = 14
ROW_X = (85.0 + np.arange(ROWS) * 160.0 / (ROWS - 1)).astype(np.float32)
CFG = R.RecoConfig(row_x=ROW_X)


def listed():
    return [
        # one sector, 200 tracks: the smallest call, made of launches and latency
        {"name": "sector", "kind": "reconstruct", "form": "staged", "sectors": 1, "tracks": 200, "frames": 1},
        # one central event of the whole detector: what one triggered event costs
        {"name": "event", "kind": "reconstruct", "form": "staged", "sectors": 36, "tracks": 10000, "frames": 1},
        # many uneven frames in one call, captured once and replayed: bulk processing
        {"name": "batch", "kind": "reconstruct", "form": "graph", "sectors": 36, "tracks": 20000, "frames": 64},
        # 50 overlapping collisions in the drift window: the continuous readout, the largest call
        {"name": "continuous", "kind": "reconstruct", "form": "staged", "sectors": 36, "tracks": 500000,
         "frames": 1, "collisions": 50},
        # forward and backward of the calibration: chi2 sum and its gradient to the distortion map
        {"name": "gradient", "kind": "gradient", "sectors": 36, "tracks": 100000, "frames": 1},
        # final fit with material and the smoothed state at every hit
        {"name": "smooth", "kind": "smooth", "sectors": 36, "tracks": 10000, "frames": 1},
        # a detector with 10 % missing hits: row-skipping search, seeding, fit with cluster errors
        {"name": "skip", "kind": "skip", "sectors": 36, "tracks": 10000, "frames": 1, "eff": 0.9},
        # prolongation of every seed with cluster pickup, refit, duplicates
        {"name": "follow", "kind": "follow", "sectors": 36, "tracks": 10000, "frames": 1},
        # links across sector edges, looper legs, refit of the linked chains
        {"name": "merge", "kind": "merge", "sectors": 36, "tracks": 10000, "frames": 1},
        # an event's clusters to integer arrays and entropy-coded streams
        {"name": "compress", "kind": "compress", "sectors": 36, "tracks": 10000, "frames": 1},
        # one large array through the entropy coder, and back
        {"name": "encode", "kind": "encode", "symbols": (1 << 28) - 77, "sigma": 12.0, "block": 1 << 15},
        {"name": "decode", "kind": "decode", "symbols": (1 << 28) - 77, "sigma": 12.0, "block": 1 << 15},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["reconstruct", "reconstruct", "frames", "continuous", "gradient", "smooth", "skip",
                       "follow", "merge", "compress", "encode", "decode"])
    if kind in ("encode", "decode"):
        return {"kind": kind, "symbols": _log(rng, 1000, 1 << 28), "sigma": round(rng.uniform(0.5, 150.0), 2),
                "block": rng.choice([1 << 13, 1 << 15])}
    if kind == "frames":
        return {"kind": "reconstruct", "form": rng.choice(["staged", "graph"]), "sectors": 36,
                "tracks": _log(rng, 500, 20000), "frames": rng.randint(2, 48)}
    if kind == "continuous":
        return {"kind": "reconstruct", "form": "staged", "sectors": 36, "tracks": _log(rng, 40000, 490000),
                "frames": 1, "collisions": rng.randint(10, 50)}
    if kind == "reconstruct":
        one = rng.random() < 0.4
        return {"kind": kind, "form": "staged", "sectors": 1 if one else 36,
                "tracks": _log(rng, 10, 1500) if one else _log(rng, 100, 30000), "frames": 1}
    if kind == "gradient":
        return {"kind": kind, "sectors": 36, "tracks": _log(rng, 1000, 100000), "frames": 1}
    case = {"kind": kind, "sectors": 36, "tracks": _log(rng, 300, 20000), "frames": 1}
    if kind == "skip":
        case["eff"] = round(rng.uniform(0.85, 1.0), 3)
    return case


def _tracks_of(case):
    """Tracks of each frame: evenly spread in the logarithm from 100 to the case's number."""
    F, n = case["frames"], case["tracks"]
    if F == 1:
        return [n]
    return [int(math.exp(math.log(100) + (k + 0.5) / F * math.log(n / 100))) for k in range(F)]


def _counts(case):
    """Clusters of tracks and of noise: the case's own, the same for every seed."""
    one = case["sectors"] == 1
    m = int(sum(_tracks_of(case)) * (37.0 if one else 114.0) * case.get("eff", 1.0))
    part = 0.05 if one else 0.10
    return m, int(round(part / (1 - part) * m))


def work(case):
    """Inputs read once, outputs written once; operations of the method itself
    (40 to 200 per cluster to find its neighbours by prediction, 300 per hit
    and fit pass, 900 for a gradient)."""
    kind = case["kind"]
    if kind in ("encode", "decode"):
        n = case["symbols"]
        bits = math.log2(max(case["sigma"], 0.5) * math.sqrt(2 * math.pi * math.e))
        return {"bytes": n * (4 + bits / 8), "flops": 10.0 * n}
    n = float(sum(_counts(case)))
    dense = case.get("collisions", 1) > 1
    hits = n * (0.32 if dense else 0.62 if kind == "gradient" else 0.88)
    seeds = n / (25 if dense else 20 if kind == "gradient" else 48)
    if kind == "reconstruct":
        return {"bytes": 16 * n + 12 * hits + 112 * seeds, "flops": (200 if dense else 40) * n + 300 * hits}
    if kind == "gradient":
        return {"bytes": 16 * hits + 200 * seeds, "flops": 1200 * hits}
    if kind == "smooth":
        return {"bytes": 93 * hits + 112 * seeds, "flops": 1500 * hits}
    if kind == "skip":
        return {"bytes": 24 * n + 13 * hits + 112 * seeds, "flops": 100 * n + 300 * hits}
    if kind == "follow":
        return {"bytes": 8 * n + 4 * hits + (112 + 4 * ROWS) * seeds, "flops": 900 * hits}
    if kind == "merge":
        return {"bytes": 12 * hits + 400 * seeds, "flops": 300 * hits + 20000 * seeds}
    return {"bytes": 8 * n + 4 * ROWS * seeds + 20 * n, "flops": 100 * n}


# ---------------------------------------------------------------------------
# inputs


def _crossings(q, ipt, phi0, tgl, nmax, sectors):
    """(track, sector, row, y, z) of every crossing of a pad-row plane, float64."""
    xr = torch.tensor(ROW_X.astype(np.float64), device=DEV)
    alpha = torch.tensor([0.0] if sectors == 1 else [(k + 0.5) * math.radians(20.0) for k in range(18)],
                         dtype=torch.float64, device=DEV)
    parts = []
    step = max(1, 30_000_000 // (alpha.numel() * ROWS))
    for c0 in range(0, q.numel(), step):
        sl = slice(c0, c0 + step)
        ph, tg = phi0[sl], tgl[sl]
        kap = -C_LIGHT * 0.5 * q[sl] * ipt[sl]
        rc = 1.0 / kap.abs()
        cx, cy = -torch.sin(ph) / kap, torch.cos(ph) / kap
        th0 = torch.atan2(-cy, -cx)
        loop = 2.0 * rc < R_OUTER
        exit_ = torch.where(loop, math.inf, 2.0 * torch.asin((R_OUTER * kap.abs() / 2).clamp(max=1.0)) / kap.abs())
        ca, sa = torch.cos(alpha), torch.sin(alpha)
        d = (cx[:, None] * ca + cy[:, None] * sa)[:, :, None] - xr
        h = torch.sqrt(rc[:, None, None] ** 2 - d * d)         # nan where the plane is not reached
        yc = (cy[:, None] * ca - cx[:, None] * sa)[:, :, None]
        for sgn in (1.0, -1.0):
            t, s, r = torch.nonzero((yc + sgn * h).abs() <= xr * TAN10, as_tuple=True)
            dk, hk = d[t, s, r], sgn * h[t, s, r]
            y = yc[t, s, 0] + hk
            th = torch.atan2(-dk * sa[s] + hk * ca[s], -dk * ca[s] - hk * sa[s])
            arc0 = rc[t] * torch.remainder(torch.where(kap[t] > 0, th - th0[t], th0[t] - th), 2 * math.pi)
            for turn in range(3):
                arc = arc0 + turn * 2 * math.pi * rc[t]
                z = tg[t] * arc
                ok = (arc <= exit_[t]) & (z.abs() <= DRIFT)
                if turn:
                    ok &= loop[t]
                k = torch.nonzero(ok)[:, 0]
                sec = s[k] if sectors == 1 else s[k] + 18 * (tg[t[k]] < 0)
                parts.append((t[k] + c0, sec, r[k], arc[k], y[k], z[k]))
        del d, h
    track, sec, row, arc, y, z = (torch.cat(v) for v in zip(*parts))
    del parts
    o = torch.argsort(arc)
    o = o[torch.argsort(track[o], stable=True)]
    first = torch.cumsum(torch.bincount(track, minlength=q.numel()), 0).roll(1)
    first[0] = 0
    rank = torch.arange(o.numel(), device=DEV) - first[track[o]]
    o = o[rank < nmax[track[o]]]
    return track[o], sec[o], row[o], y[o], z[o]


def _frames(case, seed):
    """The case's clusters: offsets (host), y, z (device float32), errors per cluster or None."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    S, F = case["sectors"], case["frames"]
    m, k = _counts(case)

    def u(k, lo=0.0, hi=1.0):
        return lo + (hi - lo) * torch.rand(k, generator=g, device=DEV, dtype=torch.float64)

    # more tracks than needed, in random order over the frames: the first m of their clusters are kept
    size = torch.tensor(_tracks_of(case), device=DEV)[torch.randperm(F, generator=g, device=DEV)]
    size = size + size // 20 + 3 * size.double().sqrt().ceil().long() + 10
    frame = torch.repeat_interleave(torch.arange(F, device=DEV), size)
    n = frame.numel()
    frame = frame[torch.randperm(n, generator=g, device=DEV)]
    q = torch.where(u(n) < 0.5, -1.0, 1.0).double()
    ipt = u(n, 0.2, 5.0)
    nmax = torch.full((n,), 1 << 30, device=DEV)
    if S > 1:                                              # loopers, truncated tracks
        ipt = torch.where(u(n) < 0.08, u(n, 1 / 0.3, 1 / 0.07), ipt)
        nmax = torch.where(u(n) < 0.5, torch.randint(5, ROWS + 1, (n,), generator=g, device=DEV), nmax)
    lim = math.radians(10.0)
    phi0 = u(n, -lim, lim) if S == 1 else u(n, 0.0, 2 * math.pi)
    tgl = u(n, -1.0, 1.0)
    coll = case.get("collisions", 1)
    track, sec, row, y, z = _crossings(q, ipt, phi0, tgl, nmax, S)
    zmax = DRIFT
    if coll > 1:                                           # collision times shift z
        t0 = u(coll, 0.0, 100.0)[torch.arange(n, device=DEV) % coll]
        z = z + torch.where(z < 0, -V_DRIFT, V_DRIFT) * t0[track]
        zmax += V_DRIFT * 100.0
    if case.get("eff", 1.0) < 1.0:
        kept = u(track.numel()) < case["eff"]
        track, sec, row, y, z = (v[kept] for v in (track, sec, row, y, z))
    track, sec, row, y, z = (v[:m] for v in (track, sec, row, y, z))
    k += m - track.numel()
    m = track.numel()
    frame = frame[track]
    if case["kind"] == "gradient":                         # distortions to be calibrated away
        amp, ph = u(S * 2, 0.0, 0.5).view(S, 1, 2), u(S * 2, 0.0, 2 * math.pi).view(S, 1, 2)
        r = torch.arange(ROWS, device=DEV)[None, :, None]
        dist = (amp * torch.sin(2 * math.pi * r / 38.0 + ph)).float().double()
        y, z = y + dist[sec, row, 0], z + dist[sec, row, 1]
    fac = torch.ones(m, 2, device=DEV, dtype=torch.float64)
    if case["kind"] == "skip":
        fac = u(2 * m, 0.5, 2.0).view(m, 2)
    noise = torch.randn(2, m, generator=g, device=DEV, dtype=torch.float64)
    y, z = y + 0.05 * fac[:, 0] * noise[0], z + 0.06 * fac[:, 1] * noise[1]
    ns = torch.randint(0, S, (k,), generator=g, device=DEV)
    nr = torch.randint(0, ROWS, (k,), generator=g, device=DEV)
    nf = torch.randint(0, F, (k,), generator=g, device=DEV)
    ny = u(k, -1.0, 1.0) * torch.tensor(ROW_X, device=DEV).double()[nr] * TAN10
    nz = u(k, -zmax, zmax) if S == 1 else torch.where(ns < 18, 1.0, -1.0) * u(k, 0.0, zmax)
    key = torch.cat([(frame * S + sec) * ROWS + row, (nf * S + ns) * ROWS + nr])
    y, z = torch.cat([y, ny]).float(), torch.cat([z, nz]).float()
    perm = torch.randperm(key.numel(), generator=g, device=DEV)
    o = perm[torch.argsort(key[perm], stable=True)]
    off = np.zeros(F * S * ROWS + 1, np.int64)
    off[1:] = np.cumsum(torch.bincount(key, minlength=off.size - 1).cpu().numpy())
    err = None
    if case["kind"] == "skip":
        fac = torch.cat([fac, torch.ones(k, 2, device=DEV, dtype=torch.float64)])[o]
        err = (fac * torch.tensor([0.05, 0.06], device=DEV, dtype=torch.float64)).float().contiguous()
    return off, y[o].contiguous(), z[o].contiguous(), err


def _map(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 7919)
    return 0.05 * torch.randn(case["sectors"], ROWS, 2, generator=g, device=DEV)


def _symbols(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return torch.randn(case["symbols"], generator=g, device=DEV).mul_(case["sigma"]).round_().int()


def _zero(obj):
    """Output buffers start at zero, so that what a pass leaves alone is the same everywhere."""
    for t in (obj.values() if isinstance(obj, dict) else vars(obj).values()):
        if isinstance(t, torch.Tensor):
            t.zero_()
    return obj


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("encode", "decode"):
        x = _symbols(case, seed)
        n, B = x.numel(), case["block"]
        st = {"case": case, "x": x, "ws": R.rans_workspace(n, RANS_L, B, DEV),
              "out": torch.zeros(R.rans_max_bytes(n, 4096, RANS_L, B), dtype=torch.uint8, device=DEV),
              "size": torch.zeros(1, dtype=torch.int64, device=DEV),
              "status": torch.zeros(1, dtype=torch.int32, device=DEV)}
        if kind == "decode":
            R.rans_encode(x, RANS_L, B, st["out"], st["ws"], st["size"], st["status"])
            size = int(st["size"].item())
            st = {"case": case, "stream": st["out"][:size].clone(), "size": size,
                  "out": torch.zeros(n, dtype=torch.int32, device=DEV)}
        return st
    cfg = CFG if case["sectors"] == 36 else R.RecoConfig(row_x=ROW_X, n_sectors=case["sectors"])
    rec = R.Reco(cfg, DEV)
    off, y, z, err = _frames(case, seed)
    fr = R.DeviceFrames(torch.from_numpy(off.astype(np.int32)).to(DEV), y, z, case["frames"], off)
    st = {"case": case, "reco": rec, "frames": fr}
    if kind == "reconstruct" and case["form"] == "graph":
        g = R.ReconstructGraph(rec, fr, mode="staged")
        for t in (g.up, g.dn):
            t.zero_()
        _zero(g.seeds)
        _zero(g.tracks)
        st["graph"] = g
        return st
    n = fr.n_clusters
    up, dn = (torch.zeros(n, dtype=torch.int32, device=DEV) for _ in range(2))
    seeds = _zero(rec.alloc_seeds(fr))
    out = (up, dn, seeds, _zero(rec.alloc_tracks(seeds)))
    ws = rec.workspace(fr)
    st.update(out=out, ws=ws)
    if kind == "reconstruct":
        return st
    if kind == "skip":
        st.update(err=err, rejected=torch.zeros(max(n, 1), dtype=torch.uint8, device=DEV))
        return st
    rec.reconstruct(fr, "staged", None, out, ws)           # the seeds (and tracks) the pass starts from
    if kind == "gradient":
        st["map"] = _map(case, seed).requires_grad_(True)
    elif kind == "smooth":
        st["tracks"] = _zero(rec.alloc_tracks(seeds))
        st["n_hits"] = int(seeds.n_hits.item())
    elif kind == "merge":
        st["merge"] = _zero(rec.alloc_merge(seeds))
        st["refit"] = dict(track_id=torch.zeros_like(st["merge"]["next"]), refit=_zero(rec.alloc_tracks(seeds)),
                           loop_par=torch.zeros(seeds.frame.numel(), 4, device=DEV),
                           loop_cov=torch.zeros(seeds.frame.numel(), 10, device=DEV),
                           loop_chi2=torch.zeros(seeds.frame.numel(), device=DEV))
    else:
        st["rows"] = torch.zeros(seeds.frame.numel(), ROWS, dtype=torch.int32, device=DEV)
        st["tracks"] = _zero(rec.alloc_tracks(seeds))
        if kind == "compress":
            rec.follow(fr, seeds, GATE, MAX_MISS, st["rows"], st["tracks"], ws)
            st["ctf"] = _zero(rec.alloc_ctf(fr, seeds))
            names = [k for k in st["ctf"] if k != "counts"]
            st["sizes"] = torch.zeros(len(names), dtype=torch.int64, device=DEV)
            st["states"] = torch.zeros(len(names), dtype=torch.int32, device=DEV)
            st["jobs"] = [dict(symbols=st["ctf"][k], n_device=st["ctf"]["counts"][i:i + 1],
                               out=torch.zeros(R.rans_max_bytes(st["ctf"][k].numel(), 1 << 20, RANS_L, 1 << 13),
                                               dtype=torch.uint8, device=DEV),
                               out_size=st["sizes"][i:i + 1], status=st["states"][i:i + 1])
                          for i, k in enumerate(names)]
            st["rws"] = R.rans_batch_workspace(st["jobs"], RANS_L, 1 << 13, DEV)
    return st


def _tracks(t):
    return {"x": t.x, "par": t.par, "cov": t.cov, "chi2": t.chi2, "ndf": t.ndf, "fit_status": t.status}


def _seeds(s):
    return {"n_seeds": s.n_seeds, "n_hits": s.n_hits, "offsets": s.offsets, "hits": s.hits, "frame": s.frame,
            "sector": s.sector, "first_row": s.first_row, "status": s.status, "hit_yz": s.hit_yz}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "encode":
        out, size, status = R.rans_encode(state["x"], RANS_L, case["block"], state["out"], state["ws"],
                                          state["size"], state["status"])
        return {"stream": out, "size": size, "status": status}
    if kind == "decode":
        sym, n, status = R.rans_decode(state["stream"], state["size"], case["symbols"], state["out"])
        return {"symbols": sym, "n": n, "status": status}
    if "graph" in state:
        up, dn, seeds, tracks = state["graph"].replay()
        return {"up": up, "dn": dn, **_seeds(seeds), **_tracks(tracks)}
    rec, fr, ws = state["reco"], state["frames"], state["ws"]
    up, dn, seeds, tracks = state["out"]
    if kind == "reconstruct":
        rec.reconstruct(fr, "staged", None, state["out"], ws)
        return {"up": up, "dn": dn, **_seeds(seeds), **_tracks(tracks)}
    if kind == "skip":
        rec.neighbours_skip(fr, up, dn, ws)
        rec.seed(fr, up, dn, seeds, ws)
        rec.fit_rows(fr, seeds, state["err"], None, tracks, state["rejected"], ws)
        return {"up": up, "dn": dn, **_seeds(seeds), **_tracks(tracks), "rejected": state["rejected"]}
    if kind == "gradient":
        state["map"].grad = None
        loss = R.KalmanChi2.apply(state["map"], rec, fr, seeds)
        loss.backward()
        return {"loss": loss, "grad": state["map"].grad}
    if kind == "smooth":
        t, rejected, par, cov = rec.smooth(fr, seeds, material=(X0, PION, CUT) + GAS, tracks=state["tracks"], ws=ws)
        par[state["n_hits"]:] = 0                              # undefined behind the last hit
        cov[state["n_hits"]:] = 0
        return {**_tracks(t), "rejected": rejected, "hit_par": par, "hit_cov": cov}
    if kind == "follow":
        rows, t = rec.follow(fr, seeds, GATE, MAX_MISS, state["rows"], state["tracks"], ws)
        return {"rows": rows, **_tracks(t)}
    if kind == "merge":
        nxt, prv, chi, mp, mc, leg, lchi = rec.merge(seeds, tracks, MERGE_CUT, state["merge"])
        f = rec.refit(fr, seeds, tracks, nxt, prv, leg, None, state["refit"])
        return {"next": nxt, "prev": prv, "link_chi2": chi, "merged_par": mp, "merged_cov": mc, "leg": leg,
                "leg_chi2": lchi, "track_id": f["track_id"], "loop_par": f["loop_par"], "loop_cov": f["loop_cov"],
                "loop_chi2": f["loop_chi2"], **_tracks(f["refit"])}
    arr = rec.ctf_build(fr, seeds, state["rows"], state["tracks"], CTF_Q, CTF_Q, state["ctf"], ws)
    jobs = R.rans_encode_batch(state["jobs"], RANS_L, 1 << 13, state["rws"])
    return {"arrays": dict(arr), "streams": [j["out"] for j in jobs], "sizes": state["sizes"],
            "states": state["states"]}


# ---------------------------------------------------------------------------
# the same in plain torch


class _Plain:
    """Clusters with their segment numbers, and the plain search and seeding on them."""

    def __init__(self, case, seed):
        self.off, self.y, self.z, self.err = _frames(case, seed)
        self.S, self.F, self.N = case["sectors"], case["frames"], self.y.numel()
        cnt = torch.from_numpy(np.diff(self.off)).to(DEV)
        self.offs = torch.from_numpy(self.off).to(DEV)
        self.seg = torch.repeat_interleave(torch.arange(cnt.numel(), device=DEV), cnt)
        self.row = self.seg % ROWS
        self.key = self.seg.double() * 4096.0 + self.y.double()
        self.order = torch.argsort(self.key)
        self.key = self.key[self.order]

    def _pairs(self, h, rows, wy, wz):
        """(index into h, cluster) pairs within the window, `rows` rows away."""
        r = self.row[h] + rows
        mid = (self.seg[h] + rows).double() * 4096.0 + self.y[h].double()
        lo = torch.searchsorted(self.key, mid - wy - 1e-3)
        n = torch.searchsorted(self.key, mid + wy + 1e-3, right=True) - lo
        n = torch.where((r >= 0) & (r < ROWS), n, 0)
        i = torch.repeat_interleave(torch.arange(h.numel(), device=DEV), n)
        at = torch.arange(i.numel(), device=DEV) - (torch.cumsum(n, 0) - n)[i] + lo[i]
        c = self.order[at]
        ok = ((self.y[c] - self.y[h[i]]).abs() <= wy) & ((self.z[c] - self.z[h[i]]).abs() <= wz)
        return i[ok], c[ok]

    def _best(self, h, spans):
        """Best (up, dn) of the clusters h over the row distances `spans`."""
        up, dn = torch.full_like(h, -1), torch.full_like(h, -1)
        Q, U, D, H = [], [], [], []
        for a, b in spans:
            iu, u = self._pairs(h, b, 2.5 * b, 2.5 * b)
            idn, d = self._pairs(h, -a, 2.5 * a, 2.5 * a)
            nd = torch.bincount(idn, minlength=h.numel())
            n = nd[iu]
            k = torch.repeat_interleave(torch.arange(iu.numel(), device=DEV), n)
            at = torch.arange(k.numel(), device=DEV) - (torch.cumsum(n, 0) - n)[k] + (torch.cumsum(nd, 0) - nd)[iu[k]]
            i, u, d = iu[k], u[k], d[at]
            g = float(np.float32(2.0) / np.float32(a + b))
            v = []
            for c in (self.y, self.z):
                e = (c[u] - c[h[i]]) / b - (c[h[i]] - c[d]) / a
                v.append(e if a + b == 2 else e * torch.tensor(g, dtype=torch.float32, device=DEV))
            ok = (v[0].abs() <= 0.6) & (v[1].abs() <= 0.75)
            q = v[0] * v[0] + v[1] * v[1]
            Q.append(q[ok]), U.append(u[ok]), D.append(d[ok]), H.append(i[ok])
        q, u, d, i = (torch.cat(v) for v in (Q, U, D, H))
        v = [q, u, d]
        for j, big in enumerate((math.inf, 1 << 40, 1 << 40)):      # smallest q, then u, then d
            best = torch.full((h.numel(),), big, dtype=v[j].dtype, device=DEV).scatter_reduce(0, i, v[j], "amin")
            k = v[j] == best[i]
            v, i = [w[k] for w in v], i[k]
        _, u, d = v
        up[i], dn[i] = u, d
        return up, dn

    def links(self, skip=False):
        up = torch.full((self.N,), -1, dtype=torch.long, device=DEV)
        dn = up.clone()
        per = max(1.0, 5.0 / 58.0 * self.N / (self.off.size - 1))      # clusters in a y window
        step = int(min(2_000_000, 60_000_000 / per)) + 1
        for spans in ([(1, 1)], [(1, 2), (2, 1)], [(2, 2)]) if skip else ([(1, 1)],):
            todo = torch.nonzero(up < 0)[:, 0]
            for c in range(0, todo.numel(), step):
                h = todo[c:c + step]
                up[h], dn[h] = self._best(h, spans)
        return up, dn

    def seeds(self, up, dn, min_hits=5):
        ids = torch.arange(self.N, device=DEV)
        lup = torch.where((up >= 0) & (dn[up.clamp(min=0)] == ids), up, -1)
        ldn = torch.where((dn >= 0) & (up[dn.clamp(min=0)] == ids), dn, -1)
        far, dist = torch.where(ldn >= 0, ldn, ids), (ldn >= 0).long()
        for _ in range(8):
            dist = dist + dist[far]
            far = far[far]
        chain = (lup >= 0) | (ldn >= 0)
        size = torch.bincount(far[chain], minlength=self.N)
        top = ids.clone()
        e = chain & (lup < 0)
        top[far[e]] = ids[e]
        b = torch.nonzero(chain & (ldn < 0))[:, 0]
        m = size[b]
        key = (((1 << 31) - m) << 32) | b
        claim = torch.full((self.N,), (1 << 63) - 1, device=DEV)
        ends, won = (dn[b], up[top[b]]), []
        may = [(v >= 0) & ~chain[v.clamp(min=0)] & (m >= min_hits - 2) for v in ends]
        for v, ok in zip(ends, may):
            claim.scatter_reduce_(0, v[ok], key[ok], "amin")
        won = [ok & (claim[v.clamp(min=0)] == key) for v, ok in zip(ends, may)]
        n = m + won[0] + won[1]
        first = torch.where(won[0], ends[0], b)
        k = torch.nonzero(n >= min_hits)[:, 0]
        k = k[torch.argsort(first[k])]
        b, n, first, w0, w1, e0, e1 = (v[k] for v in (b, n, first, won[0], won[1], ends[0], ends[1]))
        off = torch.cumsum(n, 0) - n
        hits = torch.zeros(int(n.sum()), dtype=torch.long, device=DEV)
        of = torch.full((self.N,), -1, dtype=torch.long, device=DEV)
        of[b] = torch.arange(b.numel(), device=DEV)
        i = torch.nonzero(chain & (of[far] >= 0))[:, 0]
        s = of[far[i]]
        hits[off[s] + w0[s] + dist[i]] = i
        hits[off[w0]] = e0[w0]
        hits[(off + n - 1)[w1]] = e1[w1]
        return hits, off, n, self.seg[first]


def _padded(pl, hits, off, n, sel, cap=None, corr=None):
    """Planes, y, z and errors of the hits of the seeds `sel`, [nmax, T] by hit index."""
    k = torch.arange(int(n[sel].max()), device=DEV)[:, None]
    at = (off[sel] + k.clamp(max=10 ** 9)).clamp(max=hits.numel() - 1)
    at = torch.where(k < n[sel], at, off[sel])
    h = hits[at]
    x = torch.tensor(ROW_X, device=DEV).double()[pl.row[h]]
    y, z = pl.y[h].double(), pl.z[h].double()
    if corr is not None:
        sec = (pl.seg[h] // ROWS) % pl.S
        y, z = y - corr[sec, pl.row[h], 0], z - corr[sec, pl.row[h], 1]
    s0 = torch.tensor([0.05, 0.06]).double()
    v = [(pl.err[h, i].double() ** 2) if pl.err is not None else torch.full_like(y, float(np.float32(s0[i])) ** 2)
         for i in range(2)]
    return x, y, z, v[0], v[1]


KB = -C_LIGHT * 0.5
MAX_SIN = float(np.float32(0.999))


def _asin_over(u):
    small = u.abs() < 1e-2
    w = torch.where(small, 0.5, u)
    v = u * u
    return torch.where(small, 1 + v * (1 / 6 + v * (3 / 40 + v * 5 / 112)), torch.asin(w) / w)


def _dasin_over(u):
    small = u.abs() < 1e-2
    w = torch.where(small, 0.5, u)
    v = u * u
    return torch.where(small, u * (1 / 3 + v * (3 / 10 + v * 15 / 56)),
                       (w / torch.sqrt(1 - w * w) - torch.asin(w)) / (w * w))


def _step(p, dx):
    """Helix step of p [5, T] by dx: state, Jacobian entries, whether the direction stays legal."""
    y, z, s, t, w = p
    kap = KB * w
    s2 = s + kap * dx
    ok = (s.abs() < MAX_SIN) & (s2.abs() < MAX_SIN)
    c1, c2 = torch.sqrt(1 - s * s), torch.sqrt(1 - s2 * s2)
    den = c1 + c2
    T = (s + s2) / den
    sgn = torch.where(dx < 0, -1.0, 1.0)
    sq = torch.sqrt(1 + T * T)
    chord = dx.abs() * sq
    u = kap * chord / 2
    arc = sgn * chord * _asin_over(u)
    d1, d2 = (den + (s + s2) * s / c1) / den ** 2, (den + (s + s2) * s2 / c2) / den ** 2
    ts, tw = d1 + d2, d2 * dx * KB
    q = sgn / torch.sqrt(1 - u * u) * dx.abs() * T / sq
    J = (dx * ts, dx * tw, t * q * ts, arc, t * (q * tw + sgn * chord ** 2 / 2 * _dasin_over(u) * KB), dx * KB)
    return torch.stack([y + dx * T, z + t * arc, s2, t, w]), J, ok


def _carry(J, M):
    """J M for the step's Jacobian, M [5, ..., T]."""
    f02, f04, f12, f13, f14, f24 = J
    return torch.stack([M[0] + f02 * M[2] + f04 * M[4], M[1] + f12 * M[2] + f13 * M[3] + f14 * M[4],
                        M[2] + f24 * M[4], M[3], M[4]])


def _around(J, C):
    return _carry(J, _carry(J, C).transpose(0, 1))


def _update(p, C, my, mz, vy, vz):
    r0, r1 = my - p[0], mz - p[1]
    s00, s01, s11 = C[0, 0] + vy, C[0, 1], C[1, 1] + vz
    det = s00 * s11 - s01 * s01
    a, b, c = s11 / det, -s01 / det, s00 / det
    k0, k1 = C[:, 0] * a + C[:, 1] * b, C[:, 0] * b + C[:, 1] * c
    chi = r0 * (a * r0 + b * r1) + r1 * (b * r0 + c * r1)
    return p + k0 * r0 + k1 * r1, C - k0[:, None] * C[0][None] - k1[:, None] * C[1][None], chi, det


def _start(x, y, z, n):
    T = torch.arange(n.numel(), device=DEV)
    a, b = n - 1, (n - 1) // 2
    xa, ya, za, xb, yb = x[a, T], y[a, T], z[a, T], x[b, T], y[b, T]
    xc, yc, zc = x[0], y[0], z[0]
    lbc, lab, lac = (torch.sqrt(i * i + j * j) for i, j in
                     ((xb - xc, yb - yc), (xa - xb, ya - yb), (xa - xc, ya - yc)))
    k = 2 * ((xb - xc) * (ya - yb) - (yb - yc) * (xa - xb)) / (lbc * lab * lac)
    ok = (k * lab / 2).abs().maximum((k * lac / 2).abs()) < 1
    phi = torch.atan2(ya - yb, xa - xb) + torch.asin(torch.where(ok, k * lab / 2, 0.0))
    s = torch.sin(phi)
    ok = ok & (torch.cos(phi) > 0) & (s.abs() < MAX_SIN)
    return torch.stack([ya, za, s, (za - zc) / (lac * _asin_over(torch.where(ok, k * lac / 2, 0.0))), -k / (C_LIGHT * 0.5)]), ok


def _cov0(vy, vz):
    C = torch.zeros(5, 5, vy.numel(), dtype=torch.float64, device=DEV)
    C[0, 0], C[1, 1], C[2, 2], C[3, 3], C[4, 4] = vy, vz, 1.0, 1.0, 100.0
    return C


def _gas(p, dx, sign):
    """Scattering terms, mean energy loss (new q/pT, its derivatives) and straggling of a segment."""
    s, t, w = p[2], p[3], p[4]
    t2 = 1 + t * t
    ds = dx.abs() * torch.sqrt(t2) / torch.sqrt(1 - s * s)
    x0, m, _, rho, zoa, exc = (float(np.float32(v)) for v in (X0, PION, CUT) + GAS)
    P = torch.sqrt(t2) / w.abs()
    E = torch.sqrt(P * P + m * m)
    th = 0.0136 / (P * P / E) * torch.sqrt(ds / x0) * (1 + 0.038 * torch.log(ds / x0))
    th = th * th
    Q = torch.zeros(5, 5, w.numel(), dtype=torch.float64, device=DEV)
    Q[2, 2], Q[3, 3], Q[4, 4] = th * (1 - s * s) * t2, th * t2 * t2, th * t * t * w * w
    Q[3, 4] = Q[4, 3] = th * t * w * t2
    K, me = 0.307075e-3, 0.51099895e-3
    b2, bg2 = P * P / (E * E), P * P / (m * m)
    W = 2 * me * bg2 / (1 + 2 * E / m * me / m + (me / m) ** 2)
    loss = ds * rho * K * zoa / b2 * (0.5 * torch.log(2 * me * bg2 * W / exc ** 2) - b2)
    E1 = E + sign * loss
    stop = ~(E1 > m)
    P1 = torch.sqrt((E1 * E1 - m * m).clamp(min=1e-30))
    far = stop | ((P1 - P).abs() > 0.01 * P)
    w1 = w * P / P1
    j43 = w1 * t / t2 * (1 - E1 * P * P / (E * P1 * P1))
    vw = K * zoa * rho * ds * me * (1 - 0.5 * b2) / (1 - b2) * (w * E / (P * P)) ** 2
    return Q, torch.where(far, w, w1), torch.where(far, 0.0, j43), torch.where(far, 1.0, (P / P1) ** 3 * E1 / E), \
        torch.where(far, 0.0, vw), stop


def _lose(M, j43, j44):
    return torch.cat([M[:4], (j43 * M[3] + j44 * M[4])[None]])


def _fit(x, y, z, vy, vz, n, gas=False, grad=False, rows=False):
    """Inward filter of points [nmax, T], seeds sorted by falling length.  A failing
    seed keeps what the failing step left, like the library: the plain fit ends
    after the whole step, the fits over rows (and with material) at the helix step."""
    T = torch.arange(n.numel(), device=DEV)
    p, ok = _start(x, y, z, n)
    p = torch.where(ok, p, 0.0)
    C = _cov0(vy[n - 1, T], vz[n - 1, T])
    chi, xo = torch.zeros_like(p[0]), x[n - 1, T]
    state = torch.where(ok, 0, 1)
    rej = torch.zeros(x.shape, dtype=torch.bool, device=DEV)
    for j in range(1, int(n.max())):
        a = torch.nonzero((n > j) & (state == 0))[:, 0]
        k = n[a] - 1 - j
        pa, Ca, dx = p[:, a], C[:, :, a], x[k, a] - x[k + 1, a]
        if gas:
            Q, w1, j43, j44, vw, stop = _gas(pa, dx, 1.0)
            Ca = Ca + Q
            Ca[4, 4] += vw
            Ca = _lose(_lose(Ca, j43, j44).transpose(0, 1), j43, j44)
            pa = torch.cat([pa[:4], w1[None]])
        before = Ca
        pa, J, legal = _step(pa, dx)
        if gas:
            legal = legal & ~stop
        Ca = _around(J, Ca)
        pn, Cn, d, det = _update(pa, Ca, y[k, a], z[k, a], vy[k, a], vz[k, a])
        d = torch.where(det > 0, d, -1.0)
        if gas:
            out = d > CUT
            out &= legal
            rej[k, a] = out
            pn, Cn, d = torch.where(out, pa, pn), torch.where(out, Ca, Cn), torch.where(out, 0.0, d)
        if rows:
            pn, Cn, d = torch.where(legal, pn, pa), torch.where(legal, Cn, before), torch.where(legal, d, 0.0)
        good = legal & (d >= 0) & torch.isfinite(pn).all(0)
        if grad:
            p, C, chi = p.index_copy(1, a, pn), C.index_copy(2, a, Cn), chi.index_add(0, a, d)
        else:
            p[:, a], C[:, :, a] = pn, Cn
            chi[a] += d
        xo = xo.index_copy(0, a, torch.where(good, x[k, a], xo[a]))
        state = state.index_copy(0, a, torch.where(good, 0, torch.where(legal, 3, 2)))
    return xo, p, C, chi, state, rej


TRI = [(i, j) for i in range(5) for j in range(i + 1)]


def _by_length(n):
    return torch.argsort(n, descending=True, stable=True)


def _pack(cap, sel, xo, p, C, chi):
    def full(v, *shape):
        o = torch.zeros(cap, *shape, dtype=torch.float64, device=DEV)
        o[sel] = v
        return o

    return {"x": full(xo), "par": full(p.T, 5), "cov": full(torch.stack([C[i, j] for i, j in TRI], 1), 15),
            "chi2": full(chi), "ndf": None, "fit_status": None}


def _dense(pl):
    """Candidate pairs of the plain search."""
    return 2 * pl.N * 5.0 / 58.0 * pl.N / (pl.off.size - 1)


def _smoothed(x, y, z, vy, vz, n, p0, rej):
    """State and covariance at every plane from all hits: linear filter and
    Rauch-Tung-Striebel pass about the fit's final state p0 carried outwards."""
    nm, T = x.shape
    ref = torch.zeros(nm, 5, T, dtype=torch.float64, device=DEV)
    ref[0] = p0
    for k in range(1, nm):                                     # outermost reference state
        pn, _, _ = _step(ref[k - 1], x[k] - x[k - 1])
        pn = torch.cat([pn[:4], _gas(pn, x[k] - x[k - 1], -1.0)[1][None]])
        ref[k] = torch.where(k < n, pn, ref[k - 1])
    last = ref[n - 1, :, torch.arange(T, device=DEV)].T.clone()
    eye = torch.eye(5, dtype=torch.float64, device=DEV)[:, :, None].expand(5, 5, T)
    FJ, QS = {}, {}
    d, C = torch.zeros(5, T, dtype=torch.float64, device=DEV), None
    ds, cs = {}, {}
    vo = [v[n - 1, torch.arange(T, device=DEV)] for v in (vy, vz)]
    C = _cov0(1e4 * vo[0], 1e4 * vo[1])
    cur = last
    for k in range(nm - 1, -1, -1):
        begun = k < n - 1                                      # a step arrives here from k + 1
        if k < nm - 1:
            dx = x[k] - x[k + 1]
            dx = torch.where(begun, dx, -1.0)
            Q, w1, j43, j44, vw, _ = _gas(cur, dx, 1.0)
            Q[4, 4] += vw
            nxt, J, _ = _step(torch.cat([cur[:4], w1[None]]), dx)
            F = _carry(J, _lose(eye, j43, j44))
            FJ[k + 1], QS[k + 1] = F, Q
            Cn = _mul(_mul(F, C + Q), F.transpose(0, 1))
            d = torch.where(begun, (F * d[None]).sum(1), d)
            C = torch.where(begun, Cn, C)
            cur = torch.where(begun, nxt, cur)
        ref[k] = cur
        dn_, Cn, _, _ = _update(d, C, y[k] - cur[0], z[k] - cur[1], vy[k], vz[k])
        use = (k < n) & ~rej[k]
        d, C = torch.where(use, dn_, d), torch.where(use, Cn, C)
        ds[k], cs[k] = d, C
    sp, sc = [ref[0] + ds[0]], [cs[0]]
    d, C = ds[0], cs[0]
    for k in range(1, nm):
        F, Ck = FJ[k], cs[k]
        P = _mul(_mul(F, Ck + QS[k]), F.transpose(0, 1))
        G = torch.linalg.solve(P.permute(2, 0, 1), _mul(F, Ck).permute(2, 0, 1)).permute(2, 1, 0)
        d = ds[k] + (G * (d - (F * ds[k][None]).sum(1))[None]).sum(1)
        C = Ck + _mul(_mul(G, C - P), G.transpose(0, 1))
        sp.append(ref[k] + d)
        sc.append(C)
    return torch.stack(sp), torch.stack(sc)


def _mul(A, B):
    return (A[:, :, None] * B[None]).sum(1)


def _follow(pl, hits, off, n, seg0):
    """Prolongation with pickup: the rows' clusters of every seed."""
    T = n.numel()
    tid = torch.arange(T, device=DEV)
    rows = torch.full((ROWS, T), -1, dtype=torch.long, device=DEV)
    of = torch.repeat_interleave(tid, n)
    rows[pl.row[hits], of] = hits
    o = _by_length(n)
    xo, p, C, _, state, _ = _fit(*_padded(pl, hits, off, n, o), n[o])
    p, C = p.clone(), C.clone()
    p[:, o], C[:, :, o] = p.clone(), C.clone()
    state = state[torch.argsort(o)]
    r0 = pl.row[hits[off]]
    r1 = pl.row[hits[off + n - 1]]
    base = seg0 - seg0 % ROWS
    planes = torch.tensor(ROW_X, device=DEV).double()
    v = (float(np.float32(0.05)) ** 2, float(np.float32(0.06)) ** 2)

    def search(r, a, pa, Ca):
        lo, hi = pl.offs[base[a] + r], pl.offs[base[a] + r + 1]
        best, at = torch.full_like(pa[0], math.inf), torch.full_like(a, -1)
        s00, s01, s11 = Ca[0, 0] + v[0], Ca[0, 1], Ca[1, 1] + v[1]
        det = s00 * s11 - s01 * s01
        most = int((hi - lo).max())
        c = lo[:, None] + torch.arange(most, device=DEV)
        live = c < hi[:, None]
        c = c.clamp(max=pl.N - 1)
        q0, q1 = pl.y[c].double() - pa[0][:, None], pl.z[c].double() - pa[1][:, None]
        chi = (s11[:, None] * q0 * q0 - 2 * s01[:, None] * q0 * q1 + s00[:, None] * q1 * q1) / det[:, None]
        chi = torch.where(live, chi, math.inf)
        if most:
            best, i = chi.min(1)
            at = torch.where(best <= GATE, c.gather(1, i[:, None])[:, 0], -1)
        return at

    def extend(order, x, alive, beyond):
        miss = torch.zeros_like(n)
        for r in order:
            a = torch.nonzero(alive & beyond(r))[:, 0]
            if not a.numel():
                continue
            pa, J, legal = _step(p[:, a], planes[r] - x[a])
            Ca = _around(J, C[:, :, a])
            given = rows[r, a] >= 0
            inside = legal & (given | (pa[0].abs() <= planes[r] * TAN10))
            c = torch.where(given, rows[r, a], search(r, a, pa, Ca))
            c = torch.where(inside, c, -1)
            pn, Cn, _, _ = _update(pa, Ca, pl.y[c.clamp(min=0)].double(), pl.z[c.clamp(min=0)].double(), *v)
            took = c >= 0
            p[:, a], C[:, :, a] = torch.where(took, pn, pa), torch.where(took, Cn, Ca)
            x[a] = planes[r]
            miss[a] = torch.where(took, 0, miss[a] + 1)
            rows[r, a] = c
            alive[a] = inside & (miss[a] <= MAX_MISS)
            last[:, a] = torch.where(took, pn, last[:, a])

    good = state == 0
    last = p.clone()                                           # state at the last hit taken
    x = planes[r0].clone()
    extend(range(ROWS - 1, -1, -1), x, good.clone(), lambda r: r < r0)
    inner = torch.where(rows >= 0, torch.arange(ROWS, device=DEV)[:, None], ROWS).amin(0).clamp(max=ROWS - 1)
    h = rows[inner, tid]
    p[:] = last
    p[0], p[1] = pl.y[h].double(), pl.z[h].double()
    C[:] = _cov0(torch.full_like(p[0], v[0]), torch.full_like(p[0], v[1]))
    x = planes[inner].clone()
    # rows between the hits without a cluster are stepped over: x stays, the next step is longer
    extend(range(ROWS), x, good.clone(), lambda r: (r > inner) & ((r > r1) | (rows[r] >= 0)))
    keep = rows >= 0
    m = keep.sum(0)
    at = torch.nonzero(keep.T)
    fh = rows[at[:, 1], at[:, 0]]
    return rows, fh, torch.cumsum(m, 0) - m, m, state


def exact(case, seed):
    kind = case["kind"]
    if kind in ("merge", "compress", "encode", "decode"):
        return None        # whole numbers; merging: a chain of choices between fits that single precision stores
    pl = _Plain(case, seed)
    if _dense(pl) > 8e9:
        return None        # plain pairs of a continuous frame take minutes
    up, dn = pl.links(kind == "skip")
    hits, off, n, seg0 = pl.seeds(up, dn)
    del up, dn
    cap, o = pl.N // 5 + 1, _by_length(n)
    if kind == "gradient":
        m = _map(case, seed).double().requires_grad_(True)
        loss, step = 0.0, 30000
        for c in range(0, o.numel(), step):
            s = o[c:c + step]
            with torch.no_grad():                              # failed fits take no part
                s = s[_fit(*_padded(pl, hits, off, n, s, corr=m), n[s])[4] == 0]
            part = _fit(*_padded(pl, hits, off, n, s, corr=m), n[s], grad=True)[3].sum()
            part.backward()
            loss += float(part.detach())
        return {"loss": torch.tensor(loss, dtype=torch.float64), "grad": m.grad}
    if kind == "follow":
        rows, fh, foff, m, state = _follow(pl, hits, off, n, seg0)
        o = _by_length(m)
        xo, p, C, chi, _, _ = _fit(*_padded(pl, fh, foff, m, o), m[o])
        return {"rows": None, **_pack(cap, o, xo, p, C, chi)}
    parts = []
    H = hits.numel()
    hp = torch.zeros(pl.N, 5, dtype=torch.float64, device=DEV)
    hc = torch.zeros(pl.N, 15, dtype=torch.float64, device=DEV)
    step = 8192 if kind == "smooth" else 200000
    for c in range(0, o.numel(), step):
        s = o[c:c + step]
        pts = _padded(pl, hits, off, n, s)
        xo, p, C, chi, state, rej = _fit(*pts, n[s], gas=kind == "smooth", rows=kind in ("smooth", "skip"))
        parts.append((xo, p.T, C.permute(2, 0, 1), chi))
        if kind == "smooth":
            sp, sc = _smoothed(*pts, n[s], p, rej)
            k, t = torch.nonzero((torch.arange(sp.shape[0], device=DEV)[:, None] < n[s]) & (state == 0), as_tuple=True)
            at = off[s][t] + k
            hp[at] = sp[k, :, t]
            hc[at] = torch.stack([sc[k, i, j, t] for i, j in TRI], 1)
    xo, p, C, chi = (torch.cat(v) for v in zip(*parts))
    res = _pack(cap, o, xo, p.T, C.permute(1, 2, 0), chi)
    if kind == "smooth":
        return {**res, "rejected": None, "hit_par": hp, "hit_cov": hc}
    yz = torch.zeros(max(pl.N, 1), 2, dtype=torch.float64, device=DEV)
    yz[:H, 0], yz[:H, 1] = pl.y[hits].double(), pl.z[hits].double()
    res.update({k: None for k in ("up", "dn", "n_seeds", "n_hits", "offsets", "hits", "frame", "sector",
                                  "first_row", "status")}, hit_yz=yz)
    if kind == "skip":
        res["rejected"] = None
    return res
