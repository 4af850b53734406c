"""The scan's division of chunks over workgroups and waves: events of very many windows, and
launches of few and many events, small and large.

Tolerance: 1e-6 relative between two scans of the same seeds, which run the same FP32 steps
and distances and may only differ by the rounding order of one product sum per distance
(1 ulp of a closest-approach parameter, second order in the distance).
"""
import time

import numpy as np
import pytest

from paper_1908_01949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rk():
    from paper_1908_01949_amd import rknscan
    rknscan.load_library()
    return rknscan


def _context(rk, geo, field, evs):
    c = rk.Context(0)
    c.upload_geometry(geo); c.upload_field(field); c.upload_hits(*synth.pack_events(evs))
    return c


def _scan(rk, c, p, w, n_events):
    import torch
    n = int(np.prod(w["count"].astype(np.int64), axis=1).sum())
    out = (torch.full((n,), -1.0, dtype=torch.float64, device="cuda"),
           torch.full((n,), -1, dtype=torch.int32, device="cuda"),
           torch.full((n_events,), -7, dtype=torch.int64, device="cuda"),
           torch.full((n_events,), -1.0, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    rk.rkn_scan_windows(c.ctx, p, w, *out)
    rk.rkn_synchronize(c.ctx)
    return [x.cpu().numpy() for x in out]


def test_event_of_very_many_windows(rk, geo, ufield):
    """One-point windows, a chunk each: four times as many take about four times as long
    (finding a chunk's window does not walk over the event's other windows), and each seed
    gets the score it has in a list of seeds."""
    ev = synth.event_multi_turn(geo, ufield, 3)
    c = _context(rk, geo, ufield, [ev])
    p = rk.make_scan_params(n_steps=8, precision=32, ptr_flags=rk.RKN_PTR_DEVICE)
    rng = np.random.default_rng(1)
    w = np.zeros(200000, synth.WINDOW_DTYPE)
    w["center"] = np.asarray(ev.truth_seeds[0]) + [0.05, 60, 6, 6, 6] * rng.uniform(-1, 1, (w.size, 5))
    w["count"] = 1
    took = []
    for n in (50000, 200000):
        reps = []
        for _ in range(3):
            t = time.perf_counter()
            score, nin, bi, bs = _scan(rk, c, p, w[:n], 1)
            reps.append(time.perf_counter() - t)
        took.append(min(reps))
    assert took[1] <= 8 * took[0], took      # linear: 4; a walk over the windows: 16
    q = rk.make_scan_params(n_steps=8, precision=32)
    ref = (np.zeros(w.size), np.zeros(w.size, np.int32), np.zeros(1, np.int64), np.zeros(1))
    rk.rkn_scan_seeds(c.ctx, q, np.zeros(w.size, np.int32), w["center"], *ref)
    assert np.all(np.abs(score - ref[0]) <= 1e-6 * ref[0] + 1e-6) and np.abs(nin - ref[1]).max() <= 1
    assert bi[0] == int(np.argmin(score)) and bs[0] == score.min()
    c.close()


@pytest.mark.parametrize("fieldname", ["u", "s"])
@pytest.mark.parametrize("n_events,per,count", [(2, 1, [13, 9, 15, 17, 23]), (41, 2, [5, 9, 7, 5, 7]),
                                                (30, 3, [4, 5, 4, 3, 5]), (600, 2, [3, 3, 3, 2, 2]),
                                                (3500, 1, [2, 2, 2, 2, 3])])
def test_events_shared_over_workgroups(rk, geo, ufield, sfield, fieldname, n_events, per, count):
    """Every seed is scored, as in a launch of few chunks: two events of more chunks than the
    chip has waves, 41 of some 400, 30 of 80 (at most one chunk per wave: tiles), 600 of 5
    (tiles where four-wave workgroups outnumber the events, else chunk by chunk) and 3500 of
    one or two; remainders at every window, and every third event without windows."""
    field = ufield if fieldname == "u" else sfield
    kinds = [synth.event_multi_turn(geo, ufield, 3 + k) for k in range(min(n_events, 5))]
    evs = [kinds[k % len(kinds)] for k in range(n_events)]
    c = _context(rk, geo, field, evs)
    used = [k for k in range(n_events) if n_events < 10 or k % 3 != 2]
    w = np.zeros(len(used) * per, synth.WINDOW_DTYPE)
    w["event"] = np.repeat(used, per)
    w["candidate"] = np.tile(np.arange(per), len(used))
    w["center"] = [evs[k].truth_seeds[0] for k in w["event"]]
    w["half_width"] = [0.1, 80, 8, 8, 30]
    w["count"] = count
    w["count"][:, 0] += w["candidate"]
    w["count"][:, 2] += w["event"] % 3
    size = np.prod(w["count"].astype(np.int64), axis=1)
    p = rk.make_scan_params(n_steps=90, precision=32, ptr_flags=rk.RKN_PTR_DEVICE)
    score, nin, bi, bs = _scan(rk, c, p, w, n_events)
    assert np.all(nin >= 0) and np.all(score >= 0)
    start = np.concatenate([[0], np.cumsum(size)])
    q = rk.make_scan_params(n_steps=90, precision=32)
    rng = np.random.default_rng(n_events)
    for i in (range(w.size) if w.size < 100 else rng.choice(w.size, 60, replace=False)):
        grid = [np.linspace(a - h, a + h, m) for a, h, m in zip(w[i]["center"], w[i]["half_width"], w[i]["count"])]
        at = np.sort(rng.choice(size[i], min(int(size[i]), 4000), replace=False))
        seeds = np.stack([g[k] for g, k in zip(grid, np.unravel_index(at, w[i]["count"]))], -1)
        few = (np.zeros(at.size), np.zeros(at.size, np.int32), np.zeros(n_events, np.int64), np.zeros(n_events))
        rk.rkn_scan_seeds(c.ctx, q, np.full(at.size, w[i]["event"], np.int32), seeds, *few)
        assert np.all(np.abs(score[start[i] + at] - few[0]) <= 1e-6 * few[0] + 1e-6), i
        assert np.abs(nin[start[i] + at] - few[1]).max() <= 1
    for j, k in enumerate(used):
        lo, hi = start[j * per], start[(j + 1) * per]
        assert bi[k] == lo + int(np.argmin(score[lo:hi])) and bs[k] == score[lo:hi].min()
    empty = np.setdiff1d(np.arange(n_events), used)
    assert np.all(bi[empty] == -1) and np.all(np.isinf(bs[empty]))
    c.close()


def test_a_launch_of_one_round_takes_one(rk, geo, ufield, sfield):
    """200 events of one window of 4 chunks have a workgroup each, as 64 such events do: the
    times are alike (half as long again allowed), where shares cut without regard to events
    make workgroups stage and scan a second event after the first."""
    ev = synth.event_multi_turn(geo, ufield, 3)
    p = rk.make_scan_params(n_steps=2000, precision=32, ptr_flags=rk.RKN_PTR_DEVICE)
    took = {}
    for n in (64, 200):
        c = _context(rk, geo, sfield, [ev] * n)
        w = synth.make_windows([(k, 0, ev.truth_seeds[0], [0.05, 60, 6, 6, 12], [3] * 5) for k in range(n)])
        took[n] = min(_timed(rk, c, p, w, n) for _ in range(8))
        c.close()
    assert took[200] <= 1.5 * took[64], took


def _timed(rk, c, p, w, n):
    import torch
    bi = torch.empty(n, dtype=torch.int64, device="cuda"); bs = torch.empty(n, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    t = time.perf_counter()
    rk.rkn_scan_windows_adaptive(c.ctx, p, rk.make_adaptive_params(), w, None, None, bi, bs)
    rk.rkn_synchronize(c.ctx)
    return time.perf_counter() - t
