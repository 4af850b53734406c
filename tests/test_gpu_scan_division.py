"""The scan's division of work over workgroups and waves: events of very many windows.

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
