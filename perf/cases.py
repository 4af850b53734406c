"""The calls a user of the seed scan makes, over the range of sizes they are made at.

Every case is one pass through public entry points of ``rknscan`` (or the autograd view
in ``refine``) on synthetic drift-chamber events: electrons traced from the target
through the 18-layer chamber, smeared drift distances, random noise hits. The kinds:

  seeds    rkn_scan_seeds: a handful of explicit seeds scored against their events (the
           smallest scan: a few waves, host arrays in and out)
  window   rkn_scan_windows: a seed window around a known track of one event (FP64 and
           FP32, uniform field and field map, with or without the turn-partition stop)
  event    one event end to end: Hough windows, their scan, the 8 best seeds
  batch    rkn_batch_launch + rkn_batch_topk: a planned batch of events (fixed or
           adaptive step size), the production path
  hough    rkn_hough_seed_windows: the seed windows of many events
  refine   inlier residuals and their gradient through the autograd function (forward
           and backward of the refinement)
  gn       rkn_refine_setup + rkn_gn_refine: Gauss-Newton on the best seeds per event
  bidir    rkn_bidirectional_common: hits common to both propagation directions
  turns    rkn_find_turns: the full turn-partition reconstruction loop
  rescan   rkn_rescan_refine: the coarse-to-fine rescans of a few events
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1908_01949_amd import flops, refine, rknscan as rk, synth, workloads

R0 = 500.0
KAPPA = 0.299792458
LAMBDA = 64.0
LAYER_REACH = 8.0        # a wire fires when the track passes within 8 mm
SIGMA = 0.2              # drift resolution, mm
BATCH_GRID_STEP = workloads.BATCH["hough"]["gran"]


# ---- the cases --------------------------------------------------------------------------

def listed():
    return [
        # scoring a few candidate tracks of one event, as an event display or a fit's
        # starting-point check does: latency
        dict(name="seeds_96_map", kind="seeds", field="map", precision=32, n_events=1, n_seeds=96, hits=150,
             steps=6000, turn_stop=0),
        # the FP64 reference scan of a one-turn track (workloads.SINGLE_TURN)
        dict(name="window_6^5_fp64", kind="window", field="uniform", precision=64, count=6, hits=40, steps=2000,
             turn_stop=0),
        # the exhaustive window of a multi-turn track (workloads.MULTI_TURN)
        dict(name="window_16^5_fp32", kind="window", field="uniform", precision=32, count=16, hits=156, steps=6000,
             turn_stop=0),
        # one triggered event in the field map (workloads.HOUGH_EVENT)
        dict(name="event_150hits_map", kind="event", count=12, hits=150, steps=6000),
        # the production batch (workloads.BATCH), and a small one with adaptive steps
        dict(name="batch_512_map", kind="batch", n_events=512, steps=6000, adaptive=0),
        dict(name="batch_64_adaptive", kind="batch", n_events=64, steps=6000, adaptive=1),
        # seeding alone, as a trigger-level filter uses it
        dict(name="hough_64", kind="hough", n_events=64),
        # the 8 best seeds per event of a batch (workloads.REFINE): gradient and Gauss-Newton
        dict(name="refine_512x8", kind="refine", n_events=512, k=8, steps=6000),
        dict(name="gn_128x8", kind="gn", n_events=128, k=8, steps=6000, iters=10),
        # the quality cut of a batch's best seeds
        dict(name="bidir_511", kind="bidir", n_events=511, steps=6000),
        # full event reconstruction (workloads.TURNS), a smaller set of events
        dict(name="turns_24", kind="turns", n_events=24, steps=6000),
        # the paper's refinement of a few events
        dict(name="rescan_3x8", kind="rescan", n_events=3, k=8, grid=6, rounds=3, steps=6000),
    ]


def draw(rng):
    """One more case of the same ranges (sizes spread over their logarithm, odd ones too)."""
    def logint(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))
    kind = rng.choice(["seeds", "seeds", "window", "window", "event", "batch", "hough", "refine", "gn", "bidir",
                       "turns", "rescan"])
    steps = rng.randint(1500, 6000)
    if kind == "seeds":
        return dict(kind=kind, field=rng.choice(["map", "uniform"]), precision=rng.choice([32, 32, 64]),
                    n_events=rng.randint(1, 6), n_seeds=logint(7, 1500), hits=rng.randint(40, 300), steps=steps,
                    turn_stop=rng.randint(0, 1))
    if kind == "window":
        prec = rng.choice([32, 32, 64])
        return dict(kind=kind, field=rng.choice(["map", "uniform"]), precision=prec,
                    count=rng.randint(3, 12 if prec == 32 else 7), hits=rng.randint(40, 300),
                    steps=steps, turn_stop=rng.randint(0, 1))
    if kind == "event":
        return dict(kind=kind, count=rng.randint(5, 12), hits=rng.randint(60, 300), steps=steps)
    if kind == "batch":
        return dict(kind=kind, n_events=logint(3, 256), steps=steps, adaptive=rng.randint(0, 1))
    if kind == "hough":
        return dict(kind=kind, n_events=logint(1, 256))
    if kind == "refine":
        return dict(kind=kind, n_events=logint(2, 512), k=rng.randint(1, 8), steps=steps)
    if kind == "gn":
        return dict(kind=kind, n_events=logint(2, 256), k=rng.randint(1, 8), steps=steps, iters=rng.randint(3, 10))
    if kind == "bidir":
        return dict(kind=kind, n_events=logint(3, 700), steps=steps)
    if kind == "turns":
        return dict(kind=kind, n_events=logint(2, 48), steps=rng.randint(4000, 6000))
    return dict(kind=kind, n_events=rng.randint(1, 5), k=rng.randint(2, 8), grid=rng.randint(4, 6),
                rounds=rng.randint(1, 4), steps=steps)


# ---- synthetic events ---------------------------------------------------------------------

@functools.lru_cache(None)
def _geometry():
    return synth.make_geometry()


@functools.lru_cache(None)
def _field(kind):
    return synth.uniform_field(1.0) if kind == "uniform" else synth.solenoid_field()


@functools.lru_cache(None)
def _nodes(kind):
    """(B_r, B_z) nodes [nz * nr][2] of the map on the device, FP64, or None for the uniform field."""
    f = _field(kind)
    if f.kind == "uniform":
        return None
    return torch.tensor(np.stack([f.br_grid, f.bz_grid], -1).reshape(-1, 2), dtype=torch.float64, device="cuda")


def _b(kind, x, y, z):
    """B at device points: 1 T along z, or bilinear in (r, z) clamped to the map's edge."""
    f = _field(kind)
    if f.kind == "uniform":
        o = torch.zeros_like(x)
        return o, o, o + f.bz
    t = _nodes(kind)
    r = torch.hypot(x, y)
    u = ((r - f.r0) * ((f.nr - 1) / (f.r1 - f.r0))).clamp(0, f.nr - 1)
    v = ((z - f.z0) * ((f.nz - 1) / (f.z1 - f.z0))).clamp(0, f.nz - 1)
    i = u.long().clamp(max=f.nr - 2)
    j = v.long().clamp(max=f.nz - 2)
    a, b = (u - i)[..., None], (v - j)[..., None]
    k = j * f.nr + i
    lo = torch.lerp(t[k], t[k + 1], a)
    hi = torch.lerp(t[k + f.nr], t[k + f.nr + 1], a)
    br, bz = torch.lerp(lo, hi, b).unbind(-1)
    q = br / r.clamp(min=1e-9)                    # B_r = 0 on the axis
    return q * x, q * y, bz


def _acc(kind, lam, x, t):
    bx, by, bz = _b(kind, x[..., 0], x[..., 1], x[..., 2])
    return lam[..., None] * torch.linalg.cross(t, torch.stack([bx, by, bz], -1))


def _trace(kind, rng, n, p_range, pz_range, path):
    """n candidate electrons from the target: (seeds [n][5] at the outward crossing of R0,
    reversed exit seeds [n][5], usable [n], points [n][path / 5 + 1][3] every 5 mm from the
    seed point on)."""
    h = 40.0
    p = rng.uniform(*p_range, n)
    pz = rng.uniform(*pz_range, n) * rng.choice([-1.0, 1.0], n)
    pz = np.clip(pz, -0.5 * p, 0.5 * p)
    pt = np.sqrt(p * p - pz * pz)
    ph, rv, pv = 2 * np.pi * rng.random(n), 100.0 * np.sqrt(rng.random(n)), 2 * np.pi * rng.random(n)

    def dev(a):
        return torch.tensor(a, dtype=torch.float64, device="cuda")
    x = dev(np.stack([rv * np.cos(pv), rv * np.sin(pv), rng.uniform(-200.0, 200.0, n)], -1))
    t = dev(np.stack([pt * np.cos(ph), pt * np.sin(ph), pz], -1) / p[:, None])
    p = dev(p)
    lam = -KAPPA / p
    xs, ts = [x], [t]
    n_before = int(1200 / h)
    for _ in range(n_before + int(path / h) + 2):
        a1 = _acc(kind, lam, x, t)
        t2 = t + 0.5 * h * a1
        a2 = _acc(kind, lam, x + 0.5 * h * t, t2)
        t3 = t + 0.5 * h * a2
        a3 = _acc(kind, lam, x + 0.5 * h * t2, t3)
        t4 = t + h * a3
        a4 = _acc(kind, lam, x + h * t3, t4)
        x, t = x + (h / 6) * (t + 2 * t2 + 2 * t3 + t4), t + (h / 6) * (a1 + 2 * a2 + 2 * a3 + a4)
        xs.append(x)
        ts.append(t)
    xs, ts = torch.stack(xs, 1), torch.stack(ts, 1)

    def at(s):
        """Cubic Hermite position and direction at path lengths s [n][m]."""
        k = (s / h).long().clamp(0, xs.shape[1] - 2)
        u = (s / h - k)[..., None]

        def pick(a, q):
            return torch.gather(a, 1, q[..., None].expand(-1, -1, 3))
        x0, x1, t0, t1 = pick(xs, k), pick(xs, k + 1), pick(ts, k) * h, pick(ts, k + 1) * h
        d = x0 - x1
        pos = x0 + u * (t0 + u * (-3 * d - 2 * t0 - t1 + u * (2 * d + t0 + t1)))
        dirn = t0 + u * (2 * (-3 * d - 2 * t0 - t1) + 3 * u * (2 * d + t0 + t1))
        return pos, dirn / dirn.norm(dim=-1, keepdim=True)

    r = xs[..., :2].norm(dim=-1)
    up = (r[:, :n_before] < R0) & (r[:, 1:n_before + 1] >= R0)
    usable = up.any(1)
    lo = up.float().argmax(1).double() * h
    hi = lo + h
    for _ in range(45):
        mid = 0.5 * (lo + hi)
        inside = at(mid[:, None])[0][:, 0, :2].norm(dim=-1) < R0
        lo, hi = torch.where(inside, mid, lo), torch.where(inside, hi, mid)
    s0 = 0.5 * (lo + hi)

    def seed_of(pos, dirn):
        return torch.cat([torch.atan2(pos[:, 1], pos[:, 0])[:, None], pos[:, 2:], p[:, None] * dirn], 1)
    seeds = seed_of(*(q[:, 0] for q in at(s0[:, None])))
    s = s0[:, None] + 5.0 * torch.arange(int(path / 5) + 1, device="cuda")
    pts, dirs = at(s)
    # the track's last way out of the chamber, time reversed
    r = pts[..., :2].norm(dim=-1)
    down = (r[:, :-1] >= R0) & (r[:, 1:] < R0)
    usable &= down.any(1)
    last = (down.long() * torch.arange(down.shape[1], device="cuda")).argmax(1)[:, None]
    w = ((R0 - r.gather(1, last)) / (r.gather(1, last + 1) - r.gather(1, last)))

    def mix(a):
        g = last[..., None].expand(-1, -1, 3)
        return (a.gather(1, g) * (1 - w[..., None]) + a.gather(1, g + 1) * w[..., None])[:, 0]
    exits = seed_of(mix(pts), -mix(dirs))
    return seeds, exits, usable, pts


def _wire_hits(pts):
    """Every (track, wire) passed within reach: arrays (track, wire, distance, chord),
    ordered by track, then along the track."""
    geo = _geometry()
    n, n_w = pts.shape[0], geo.n_wires
    a, d = pts[:, :-1], pts[:, 1:] - pts[:, :-1]
    c = a + 0.5 * d
    rc, phi = c[..., :2].norm(dim=-1), torch.atan2(c[..., 1], c[..., 0])
    wires = {k: torch.tensor(getattr(geo, k), device="cuda") for k in ("mx", "my", "mz", "ux", "uy", "uz")}
    keys, dist = [], []
    for l in range(geo.n_layers):
        band = (rc > geo.layer_rmin[l] - 12) & (rc < geo.layer_rmax[l] + 12) & (c[..., 2].abs() < geo.half_z)
        tr, ch = torch.nonzero(band, as_tuple=True)
        if tr.numel() == 0:
            continue
        nw = int(geo.layer_nwires[l])
        shift = torch.atan2(c[tr, ch, 2] * math.tan(geo.layer_stereo[l]),
                            torch.full_like(rc[tr, ch], float(geo.layer_radius[l])))
        j0 = torch.round((phi[tr, ch] - shift) * (nw / (2 * math.pi)) - 0.5 * (l % 2)).long()
        for dj in (-1, 0, 1):
            g = int(geo.layer_first[l]) + torch.remainder(j0 + dj, nw)
            m = torch.stack([wires["mx"][g], wires["my"][g], wires["mz"][g]], -1)
            u = torch.stack([wires["ux"][g], wires["uy"][g], wires["uz"][g]], -1)
            rr, dd = a[tr, ch] - m, d[tr, ch]
            rr, dd = rr - (rr * u).sum(-1, keepdim=True) * u, dd - (dd * u).sum(-1, keepdim=True) * u
            s = (-(rr * dd).sum(-1) / (dd * dd).sum(-1).clamp(min=1e-12)).clamp(0, 1)
            q = (rr + s[:, None] * dd).norm(dim=-1)
            ok = q <= LAYER_REACH
            keys.append((tr[ok] * n_w + g[ok]) * 100000 + ch[ok])
            dist.append(q[ok])
    if not keys:
        z = np.zeros(0, np.int64)
        return z, z, z.astype(float), z
    keys, dist = torch.cat(keys).cpu().numpy(), torch.cat(dist).cpu().numpy()
    order = np.lexsort((keys, dist, keys // 100000))      # per (track, wire): the closest chord first
    keys, dist = keys[order], dist[order]
    first = np.ones(keys.size, bool)
    first[1:] = keys[1:] // 100000 != keys[:-1] // 100000
    keys, dist = keys[first], dist[first]
    tw, ch = keys // 100000, keys % 100000
    order = np.lexsort((ch, tw // n_w))
    return tw[order] // n_w, tw[order] % n_w, dist[order], ch[order]


def _events(kind, seed, n_events, path, tracks=(1, 1), hits=(150, 150), noise=(0.2, 0.2), p_range=(104.97, 104.97),
            pz_range=(5.0, 20.0), min_hits=None, single_turn=False):
    """n_events events: CSR hits, and the seed and reversed exit seed of each event's first
    track. `hits`: total hits; `noise`: noise fraction; `min_hits`: true hits a track needs."""
    rng = np.random.default_rng([190801949, seed, n_events])
    geo = _geometry()
    plan = [(int(rng.integers(tracks[0], tracks[1] + 1)), int(rng.integers(hits[0], hits[1] + 1)),
             rng.uniform(*noise)) for _ in range(n_events)]
    if tracks[1] > 1:
        plan[0] = (tracks[1], hits[1], plan[0][2])      # one event is the largest of its kind
    need = sum(t for t, _, _ in plan)
    if min_hits is None:
        # a track that gives fewer true hits than asked makes a smaller event
        min_hits = 40 if tracks[1] > 1 or single_turn else min(110, int(math.ceil(hits[1] * (1 - noise[0]))))
    pool = []
    while len(pool) < need:
        seeds, exits, usable, pts = _trace(kind, rng, 2 * (need - len(pool)) + 12, p_range, pz_range, path)
        tr, w, d, _ = _wire_hits(pts)
        bounds = np.searchsorted(tr, np.arange(pts.shape[0] + 1))
        seeds, exits, usable = seeds.cpu().numpy(), exits.cpu().numpy(), usable.cpu().numpy()
        for k in range(pts.shape[0]):
            lo, hi = bounds[k], bounds[k + 1]
            if usable[k] and hi - lo >= min_hits and len(pool) < need:
                pool.append((seeds[k], exits[k], w[lo:hi], d[lo:hi]))
    off, wid, dr, first_seed, first_exit = [0], [], [], [], []
    at = 0
    for e, (nt, total, frac) in enumerate(plan):
        mine = pool[at:at + nt]
        at += nt
        # round-robin along the tracks, one hit per wire
        rank = np.concatenate([np.arange(m[2].size) for m in mine])
        ww, dd = np.concatenate([m[2] for m in mine]), np.concatenate([m[3] for m in mine])
        order = np.argsort(rank, kind="stable")
        ww, dd = ww[order], dd[order]
        _, idx = np.unique(ww, return_index=True)
        n_true = total - int(round(frac * total))
        idx = np.sort(idx)[:n_true]
        ww, dd = ww[idx], dd[idx]
        # the drawn noise fraction, also when the tracks give fewer hits than asked
        n_noise = total - ww.size if ww.size == n_true or e == 0 else int(frac / (1 - frac) * ww.size)
        free = np.setdiff1d(np.arange(geo.n_wires), ww)
        noise_w = rng.choice(free, size=n_noise, replace=False)
        drift = np.concatenate([np.clip(dd + rng.normal(0, SIGMA, dd.size), 0, LAYER_REACH),
                                rng.uniform(0, LAYER_REACH, n_noise)])
        ww = np.concatenate([ww, noise_w])
        order = np.argsort(ww, kind="stable")
        wid.append(ww[order].astype(np.int32))
        dr.append(drift[order].astype(np.float32))
        off.append(off[-1] + ww.size)
        first_seed.append(mine[0][0])
        first_exit.append(mine[0][1])
    return dict(off=np.array(off, np.int32), wire=np.concatenate(wid), drift=np.concatenate(dr),
                seed=np.array(first_seed), exit=np.array(first_exit))


def _batch_events(seed, n_events, steps):
    return _events("map", seed, n_events, steps, tracks=(1, 3), hits=(40, 300), noise=(0.1, 0.4),
                   p_range=(60.0, 105.0), pz_range=(0.0, 25.0))


def _near(rng, seeds, n, scale=(0.003, 25.0, 0.8, 0.8, 3.0)):
    """n seeds around each given one, as the best seeds of a coarse scan lie."""
    return (seeds[:, None, :] + np.array(scale) * rng.uniform(-1, 1, (seeds.shape[0], n, 5))).reshape(-1, 5)


def _inputs(case, seed):
    """The arrays a case starts from, from the seed alone."""
    kind, rng = case["kind"], np.random.default_rng([19, seed])
    steps = case.get("steps", 6000)
    if kind in ("seeds", "window", "event"):
        one_turn = kind == "window" and steps <= 2000
        ev = _events(case.get("field", "map"), seed, case.get("n_events", 1), steps,
                     hits=(case["hits"], case["hits"]), noise=(0.0, 0.0) if one_turn else (0.25, 0.25),
                     single_turn=one_turn or steps < 4000)
        if kind == "seeds":
            ne, n = case["n_events"], case["n_seeds"]
            ev["seed_event"] = np.sort(rng.integers(0, ne, n)).astype(np.int32)
            ev["seeds"] = _near(rng, ev["seed"][ev["seed_event"]], 1)
        return ev
    if kind == "turns":
        return _events("map", seed, case["n_events"], 6000, hits=(135, 135), noise=(0.23, 0.23), min_hits=104)
    ev = _batch_events(seed, case["n_events"], steps)
    if kind in ("refine", "gn"):
        ev["seed_event"] = np.repeat(np.arange(case["n_events"], dtype=np.int32), case["k"])
        ev["seeds"] = _near(rng, ev["seed"], case["k"])
        # the point the gradient is asked at: a small update away from the setup seeds
        ev["moved"] = ev["seeds"] + np.array((2e-4, 2.0, 0.05, 0.05, 0.2)) * rng.uniform(-1, 1, ev["seeds"].shape)
    if kind == "bidir":
        ev["entry"], ev["exit"] = _near(rng, ev["seed"], 1), _near(rng, ev["exit"], 1)
    if kind == "rescan":
        ev["seeds"] = _near(rng, ev["seed"], case["k"], BATCH_GRID_STEP)
    return ev


# ---- what a program holds before the call, and the call ------------------------------------------

@functools.lru_cache(None)
def _stream():
    """The one stream a program runs its contexts on."""
    return torch.cuda.Stream()


def prepare(case, seed):
    kind, steps = case["kind"], case.get("steps", 6000)
    ev = _inputs(case, seed)
    field = _field(case.get("field", "map"))
    ctx = rk.Context(0, _stream().cuda_stream)
    ctx.upload_geometry(_geometry())
    ctx.upload_field(field)
    ctx.upload_hits(ev["off"], ev["wire"], ev["drift"])
    ne = ctx.n_events
    s = dict(kind=kind, ctx=ctx, ne=ne)

    def dev(shape, dtype):
        return torch.zeros(shape, dtype=dtype, device="cuda")

    def params(**kw):
        return rk.make_scan_params(n_steps=steps, lambda_mm2=LAMBDA, turn_stop=case.get("turn_stop", 0),
                                   precision=case.get("precision", 32), **kw)
    if kind == "seeds":
        n = case["n_seeds"]
        s.update(p=params(), seed_event=ev["seed_event"], seeds=ev["seeds"],
                 out=(np.zeros(n), np.zeros(n, np.int32), np.zeros(ne, np.int64), np.zeros(ne)))
    elif kind == "window":
        w = synth.make_windows([(0, 0, ev["seed"][0], workloads.SINGLE_TURN["half_width"], [case["count"]] * 5)])
        n = case["count"] ** 5
        s.update(p=params(ptr_flags=rk.RKN_PTR_DEVICE), windows=w,
                 out=(dev(n, torch.float64), dev(n, torch.int32), dev(ne, torch.int64), dev(ne, torch.float64)))
    elif kind == "event":
        h = dict(workloads.HOUGH_EVENT["hough"], count=(case["count"],) * 5, count_max=case["count"],
                 max_seeds_window=case["count"] ** 5)
        s.update(p=params(ptr_flags=rk.RKN_PTR_DEVICE), hp=rk.make_hough_params(b_ref=field.b_ref, **h),
                 out=(dev((ne, 8), torch.int64), dev((ne, 8), torch.float64), dev((ne, 8, 5), torch.float64)))
    elif kind == "batch":
        p = params(ptr_flags=rk.RKN_PTR_DEVICE)
        hp = rk.make_hough_params(b_ref=field.b_ref, **workloads.BATCH["hough"])
        if case["adaptive"]:
            rk.rkn_batch_plan_adaptive(ctx.ctx, hp, p, rk.make_adaptive_params())
        else:
            rk.rkn_batch_plan(ctx.ctx, hp, p)
        s.update(best=(dev(ne, torch.int64), dev(ne, torch.float64)),
                 top=(dev((ne, 8), torch.int64), dev((ne, 8), torch.float64), dev((ne, 8, 5), torch.float64)))
    elif kind == "hough":
        s.update(hp=rk.make_hough_params(b_ref=field.b_ref, **workloads.BATCH["hough"]))
    elif kind == "refine":
        s.update(ref=refine.Refinement(ctx, params(), ev["seed_event"], ev["seeds"],
                                       workloads.REFINE["ckpt_every"]),
                 moved=torch.tensor(ev["moved"], device="cuda"))
    elif kind == "gn":
        n = ev["seed_event"].size
        s.update(p=params(), seed_event=ev["seed_event"], seeds=ev["seeds"], iters=case["iters"],
                 out=(np.zeros((n, 5)), np.zeros((n, case["iters"] + 1))))
    elif kind == "bidir":
        s.update(p=params(ptr_flags=rk.RKN_PTR_DEVICE), pair_event=np.arange(ne, dtype=np.int32),
                 entry=ev["entry"], exit=ev["exit"],
                 out=(dev((ne, ctx.max_hits), torch.uint8), dev((ne, ctx.max_hits), torch.uint8),
                      dev(ne, torch.int32)))
    elif kind == "turns":
        s.update(p=params(), hp=rk.make_hough_params(b_ref=field.b_ref, **workloads.TURNS["hough"]),
                 tp=rk.make_turn_params(), n_hits=int(ev["off"][-1]))
    elif kind == "rescan":
        step = np.broadcast_to(np.array(BATCH_GRID_STEP), ev["seeds"].shape).copy()
        s.update(p=params(), rp=rk.make_rescan_params(k=case["k"], grid=case["grid"], max_rounds=case["rounds"]),
                 seeds=ev["seeds"], step=step)
    return s


def run(s):
    kind, c = s["kind"], s["ctx"].ctx
    if kind == "seeds":
        return rk.rkn_scan_seeds(c, s["p"], s["seed_event"], s["seeds"], *s["out"])
    if kind == "window":
        return rk.rkn_scan_windows(c, s["p"], s["windows"], *s["out"])
    if kind == "event":
        w = rk.rkn_hough_seed_windows(c, s["hp"])
        return dict(windows=_window_arrays(w), top=rk.rkn_scan_windows_topk(c, s["p"], w, 8, *s["out"]))
    if kind == "batch":
        rk.rkn_batch_launch(c, *s["best"])
        rk.rkn_batch_topk(c, 8, *s["top"])
        return s["best"], s["top"]
    if kind == "hough":
        return _window_arrays(rk.rkn_hough_seed_windows(c, s["hp"]))
    if kind == "refine":
        x = s["moved"].clone().requires_grad_(True)
        resid = s["ref"].residuals(x)
        torch.nan_to_num(resid).square().sum().backward()
        return resid, x.grad
    if kind == "gn":
        rk.rkn_refine_setup(c, s["p"], s["seed_event"], s["seeds"], workloads.REFINE["ckpt_every"])
        return rk.rkn_gn_refine(c, s["iters"], workloads.REFINE["scale"], *s["out"])
    if kind == "bidir":
        return rk.rkn_bidirectional_common(c, s["p"], s["pair_event"], s["entry"], s["exit"], s["ctx"].max_hits,
                                           *s["out"])
    if kind == "turns":
        return rk.rkn_find_turns(c, s["hp"], s["p"], s["tp"], s["n_hits"], s["ne"])
    return rk.rkn_rescan_refine(c, s["p"], s["rp"], s["ne"], s["seeds"], s["step"])


def _window_arrays(w):
    return dict(event=w["event"], center=w["center"], half_width=w["half_width"], count=w["count"])


# ---- the least work ---------------------------------------------------------------------------------

def work(case):
    """Flops of the propagation (its steps as the method states them, in the field at hand)
    plus one chord distance per seed and hit, and each input and output once. The windows
    of a batch hold about 60 000 seeds per event."""
    kind, steps, ne = case["kind"], case.get("steps", 6000), case.get("n_events", 1)
    f = flops.F_RKN_UNIFORM if case.get("field", "map") == "uniform" else flops.F_RKN_GRID
    hits = case.get("hits", 170)
    wires = _geometry().n_wires * 64 + (65 * 129 * 8 if f == flops.F_RKN_GRID else 0) + ne * hits * 8
    votes = 256 * 256 * hits * 10

    def scan(n):
        return n * (steps * f + hits * flops.F_DOCA)
    if kind == "seeds":
        n = case["n_seeds"]
        return dict(bytes=wires + n * (44 + 12) + ne * 16, flops=scan(n))
    if kind == "window":
        n = case["count"] ** 5
        return dict(bytes=wires + n * 12, flops=scan(n))
    if kind == "event":
        n = 4 * case["count"] ** 5
        return dict(bytes=wires + 8 * 56, flops=scan(n) + votes)
    if kind == "batch":
        # an adaptive step covers about 4 mm
        return dict(bytes=wires + ne * (16 + 8 * 56),
                    flops=ne * (scan(60000) / (4 if case["adaptive"] else 1) + votes))
    if kind == "hough":
        return dict(bytes=wires + ne * 4 * 112, flops=ne * votes)
    if kind in ("refine", "gn"):
        # backward: the tangents of 5 seed parameters and the adjoint, about 6 forward steps
        n = ne * case["k"]
        passes = 1 + 6 if kind == "refine" else 2 + 7 * case["iters"]
        return dict(bytes=wires + n * (300 * 4 + 80), flops=passes * scan(n))
    if kind == "bidir":
        return dict(bytes=wires + ne * (80 + 600), flops=2 * scan(ne))
    if kind == "turns":
        # Hough windows, then about two neighbour windows per event; a turn takes ~1500 steps
        n = 4 * 7 * 13 * 7 * 7 * 13 + 2 * 5 * 9 * 5 * 5 * 9
        return dict(bytes=wires + ne * 8 * 100, flops=ne * (0.3 * scan(n) + votes))
    n = ne * case["k"] * case["grid"] ** 5
    return dict(bytes=wires + ne * case["k"] * 200, flops=case["rounds"] * scan(n))


# ---- the same results in 64 bits -----------------------------------------------------------------------

def _paths(kind, seeds, steps, turn_stop):
    """Positions [steps + 1][n][3] of the fixed-step RKN4 (h = 1 mm) in FP64."""
    s = torch.as_tensor(seeds, dtype=torch.float64, device="cuda")
    p = s[:, 2:].norm(dim=1)
    lam = -KAPPA / p
    x = torch.stack([R0 * torch.cos(s[:, 0]), R0 * torch.sin(s[:, 0]), s[:, 1]], -1)
    t = s[:, 2:] / p[:, None]
    out = torch.empty((steps + 1, *x.shape), dtype=torch.float64, device="cuda")
    out[0] = x
    live = torch.ones(x.shape[0], dtype=torch.bool, device="cuda")

    def cross(tt, b):
        return lam[:, None] * torch.linalg.cross(tt, b)

    def b(q):
        return torch.stack(_b(kind, q[:, 0], q[:, 1], q[:, 2]), -1)
    for i in range(steps):
        k1 = cross(t, b(x))
        mid = b(x + 0.5 * t + 0.125 * k1)
        k2 = cross(t + 0.5 * k1, mid)
        k3 = cross(t + 0.5 * k2, mid)
        k4 = cross(t + k3, b(x + t + 0.5 * k3))
        nx = x + t + (k1 + k2 + k3) / 6
        nt = t + (k1 + 2 * (k2 + k3) + k4) / 6
        if turn_stop:
            x, t = torch.where(live[:, None], nx, x), torch.where(live[:, None], nt, t)
            live &= x[:, :2].norm(dim=1) >= R0
        else:
            x, t = nx, nt
        out[i + 1] = x
    return out


def _segment_wire(p0, d, m, u, half):
    """Closest points of chords p0 + s d and wires m + t u, |t| <= half: (d2, s, vector)."""
    r = p0 - m
    a, b = (d * d).sum(-1), (d * u).sum(-1)
    e, f = (d * r).sum(-1), (u * r).sum(-1)
    den = a - b * b
    s = torch.where(den > 1e-12 * a, (b * f - e) / den.clamp(min=1e-300), torch.zeros_like(a)).clamp(0, 1)
    t = b * s + f
    tc = torch.maximum(torch.minimum(t, half), -half)
    s2 = torch.where(a > 0, (tc * b - e) / a.clamp(min=1e-300), torch.zeros_like(a)).clamp(0, 1)
    s = torch.where(tc != t, s2, s)
    v = r + s[..., None] * d - tc[..., None] * u
    return (v * v).sum(-1), s, v


def _event_wires(ev, e):
    geo = _geometry()
    g = ev["wire"][ev["off"][e]:ev["off"][e + 1]]

    def dev(a):
        return torch.tensor(np.asarray(a, np.float64), device="cuda")
    return (dev(np.stack([geo.mx[g], geo.my[g], geo.mz[g]], -1)), dev(np.stack([geo.ux[g], geo.uy[g], geo.uz[g]], -1)),
            dev(geo.half_len[g]), dev(ev["drift"][ev["off"][e]:ev["off"][e + 1]]))


def _closest(paths, m, u, half):
    """(D [n][H], chord [n][H]) over the chords of paths [steps + 1][n][3]."""
    n, h = paths.shape[1], m.shape[0]
    chunk = max(1, int(1.5e7 / (n * h)))
    best = torch.full((n, h), math.inf, dtype=torch.float64, device="cuda")
    arg = torch.zeros((n, h), dtype=torch.long, device="cuda")
    for i in range(0, paths.shape[0] - 1, chunk):
        q = paths[i:i + chunk + 1]
        d2 = _segment_wire(q[:-1, :, None, :], (q[1:] - q[:-1])[:, :, None, :], m, u, half)[0]
        v, k = d2.min(0)
        arg = torch.where(v < best, k + i, arg)
        best = torch.minimum(v, best)
    return best.sqrt(), arg


def _grid(center, half, count):
    axes = [np.linspace(c - w, c + w, count) for c, w in zip(center, half)]
    return np.stack([a.reshape(-1) for a in np.meshgrid(*axes, indexing="ij")], -1)


def _exact_scores(case, ev, seed_event, seeds):
    paths = _paths(case["field"], seeds, case["steps"], case["turn_stop"])
    score = torch.zeros(len(seeds), dtype=torch.float64, device="cuda")
    best = torch.full((len(ev["off"]) - 1,), math.inf, dtype=torch.float64, device="cuda")
    for e in np.unique(seed_event):
        at = torch.tensor(np.nonzero(seed_event == e)[0], device="cuda")
        m, u, half, drift = _event_wires(ev, e)
        dist, _ = _closest(paths[:, at], m, u, half)
        score[at] = ((dist - drift) ** 2).clamp(max=LAMBDA).sum(1)
        best[e] = score[at].min()
    # counts and the best index are whole numbers: equal on both sides, no 64-bit value
    return score, None, None, best


def _exact_gradient(case, ev):
    """Residuals at the moved seeds on the inlier sets of the setup seeds, and the gradient
    of the sum of their squares: each distance's derivative along its closest chord, the
    chord's by central differences of FP64 paths."""
    seeds, n = ev["moved"], len(ev["moved"])
    eps = np.array((1e-6, 1e-4, 1e-5, 1e-5, 1e-5))
    copies = [seeds] + [seeds + s * eps * (np.arange(5) == j) for j in range(5) for s in (1, -1)]
    paths = _paths("map", np.concatenate([ev["seeds"], *copies]), case["steps"], 0)
    width = int(np.diff(ev["off"]).max())
    resid = torch.full((n, width), math.nan, dtype=torch.float64, device="cuda")
    grad = torch.zeros((n, 5), dtype=torch.float64, device="cuda")
    k = case["k"]
    for e in range(case["n_events"]):
        at = slice(e * k, e * k + k)
        m, u, half, drift = _event_wires(ev, e)
        inlier = (_closest(paths[:, :n][:, at], m, u, half)[0] - drift) ** 2 < LAMBDA
        moved = paths[:, n:2 * n][:, at]
        dist, arg = _closest(moved, m, u, half)
        row = torch.arange(k, device="cuda")[:, None].expand_as(arg)
        p0, p1 = moved[arg, row], moved[arg + 1, row]
        _, s, v = _segment_wire(p0, p1 - p0, m, u, half)
        w = v / dist.clamp(min=1e-12)[..., None]
        r = torch.where(inlier, dist - drift, torch.zeros_like(dist))
        resid[at, :m.shape[0]] = torch.where(inlier, r, torch.full_like(r, math.nan))
        for j in range(5):
            hi = paths[:, (2 + 2 * j) * n:(3 + 2 * j) * n][:, at]
            lo = paths[:, (3 + 2 * j) * n:(4 + 2 * j) * n][:, at]
            dx = (1 - s)[..., None] * (hi[arg, row] - lo[arg, row]) + s[..., None] * (hi[arg + 1, row] - lo[arg + 1, row])
            grad[at, j] = (2 * r * (w * dx).sum(-1)).sum(1) / (2 * eps[j])
    return resid, grad


def _hough_peaks(hp, x, y):
    """The best peaks (count, a, b, k) of one event's vote, and its accumulator."""
    n, nr = hp.n_xy, hp.n_r
    w, wr = 2 * hp.xy_half / n, (hp.r_max - hp.r_min) / nr
    c = -hp.xy_half + w * (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5)
    q = torch.round(torch.stack([x, y]) * 256) / 256
    acc = torch.zeros(n * n * nr, dtype=torch.int32, device="cuda")
    r = torch.sqrt((c[:, None, None] - q[0]) ** 2 + (c[None, :, None] - q[1]) ** 2)
    k = torch.floor((r - hp.r_min) / wr).long()
    ok = (k >= 0) & (k < nr)
    flat = torch.arange(n * n, device="cuda").reshape(n, n, 1) * nr + k
    acc.index_add_(0, flat[ok], torch.ones_like(flat[ok], dtype=torch.int32))
    acc = acc.reshape(n, n, nr)
    thr = max(hp.min_votes, (int(acc.max()) + 1) // 2, 1)
    pad = torch.nn.functional.pad(acc, (1, 1, 1, 1, 1, 1), value=-1)
    peak = acc >= thr
    for i in range(27):
        if i == 13:
            continue
        da, db, dk = i // 9, i // 3 % 3, i % 3
        o = pad[da:da + n, db:db + n, dk:dk + nr]
        peak &= (acc > o) if i < 13 else (acc >= o)
    at = torch.nonzero(peak.reshape(-1))[:, 0]
    cnt = acc.reshape(-1)[at]
    got = sorted(zip((-cnt).tolist(), at.tolist()))[:hp.max_cand]
    return [(-v, f // (n * nr), f // nr % n, f % nr) for v, f in got], acc


def _exact_hough(ev, hp):
    geo = _geometry()
    w, wr = 2 * hp.xy_half / hp.n_xy, (hp.r_max - hp.r_min) / hp.n_r
    centers, halfs = [], []
    for e in range(len(ev["off"]) - 1):
        g = ev["wire"][ev["off"][e]:ev["off"][e + 1]]
        peaks, acc = _hough_peaks(hp, torch.tensor(geo.mx[g], device="cuda"), torch.tensor(geo.my[g], device="cuda"))
        acc = acc.cpu().numpy() if peaks else None
        for v, a, b, k in peaks:
            xc, yc, r = -hp.xy_half + w * (a + 0.5), -hp.xy_half + w * (b + 0.5), hp.r_min + wr * (k + 0.5)
            d = math.hypot(xc, yc)
            if not (0 < d <= r + R0 and d >= abs(r - R0)):
                continue
            al = (R0 * R0 - r * r + d * d) / (2 * d)
            hh = math.sqrt(max(R0 * R0 - al * al, 0.0))
            cx, cy = xc / d, yc / d
            best, pick = 0.0, None
            for px, py in ((al * cx - hh * cy, al * cy + hh * cx), (al * cx + hh * cy, al * cy - hh * cx)):
                vx, vy = -(py - yc) / r, (px - xc) / r          # an electron turns counter-clockwise
                if vx * px + vy * py > best:
                    best, pick = vx * px + vy * py, (px, py, vx, vy)
            if pick is None:
                continue
            px, py, vx, vy = pick
            pt = KAPPA * hp.b_ref * r
            centers.append([math.atan2(py, px), hp.center_z, pt * vx, pt * vy, hp.center_pz])
            extent = 1
            for line, at in ((acc[:, b, k], a), (acc[a, :, k], b), (acc[a, b, :], k)):
                lo, hi = at, at
                while lo > 0 and 2 * line[lo - 1] >= v:
                    lo -= 1
                while hi + 1 < line.size and 2 * line[hi + 1] >= v:
                    hi += 1
                extent = max(extent, hi - lo + 1)
            count = [max(1, min(hp.count_max, hp.count[q] + hp.grow[q] * (extent - 1))) for q in range(5)]
            while math.prod(count) > hp.max_seeds_window and max(count) > 1:
                count[count.index(max(count))] -= 1
            halfs.append([hp.gran[q] * 0.5 * (count[q] - 1) for q in range(5)])
    # paths of the outputs that run() returns: event and count are whole numbers
    return dict(event=None, center=np.array(centers).reshape(-1, 5), half_width=np.array(halfs).reshape(-1, 5),
                count=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "seeds":
        ev = _inputs(case, seed)
        return _exact_scores(case, ev, ev["seed_event"], ev["seeds"])
    if kind == "window" and case["count"] ** 5 * case["steps"] * case["hits"] <= 1e9:
        ev = _inputs(case, seed)
        seeds = _grid(ev["seed"][0], workloads.SINGLE_TURN["half_width"], case["count"])
        return _exact_scores(case, ev, np.zeros(len(seeds), np.int32), seeds)
    if kind == "hough":
        ev = _inputs(case, seed)
        return _exact_hough(ev, rk.make_hough_params(b_ref=_field("map").b_ref, **workloads.BATCH["hough"]))
    if kind == "refine":
        return _exact_gradient(case, _inputs(case, seed))
    # batches, Gauss-Newton, rescans and the turn loop: too many brute-force distances; the
    # two-direction masks and counts are whole numbers
    return None
