"""Selection over slices: an event's seeds are read by several workgroups when there are
few events. Index work, so compared exactly with a host sort of the same scores, at seed
counts around the slice and workgroup sizes and over event counts on both sides of the
split (one event: 256 slices; 5: 103; 512: none)."""
import numpy as np
import pytest

from paper_1908_01949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_events,counts", [
    (1, [[1, 1, 1, 1, 1]]), (1, [[5, 51, 1, 1, 1]]), (1, [[16, 16, 1, 1, 1]]), (1, [[17, 13, 7, 3, 5]]),
    (1, [[16, 16, 16, 16, 5]]), (5, [[1, 2, 3, 1, 1], [103, 1, 1, 1, 1], [8, 13, 5, 5, 5]]),
    (512, [[2, 3, 1, 1, 1], [1, 1, 17, 1, 1]])])
def test_topk_equals_a_host_sort(geo, ufield, n_events, counts):
    from paper_1908_01949_amd import rknscan as rk
    base = synth.event_single_turn(geo, ufield, 0)
    off, wid, dr = synth.pack_events([base] * n_events)
    c = rk.Context(0)
    c.upload_geometry(geo); c.upload_field(ufield); c.upload_hits(off, wid, dr)
    hw = [0.05, 20.0, 3.0, 3.0, 0.0]   # the last one repeats seeds: equal scores
    picked = [e for e in range(n_events) if n_events == 1 or e % 3 != 1]   # the others have no seeds
    w = synth.make_windows([(e, 0, base.truth_seeds[0], hw, counts[i % len(counts)]) for i, e in enumerate(picked)])
    sp = rk.make_scan_params(n_steps=200, precision=32)
    sizes = [int(np.prod(x["count"].astype(np.int64))) for x in w]
    score = np.zeros(sum(sizes))
    rk.rkn_scan_windows(c.ctx, sp, w, score, None, np.zeros(n_events, np.int64), np.zeros(n_events))
    for k in (1, 5, 16):
        idx, sc, _ = rk.rkn_scan_windows_topk(c.ctx, sp, w, k, n_events=n_events)
        want_i, want_s = np.full((n_events, k), -1, np.int64), np.full((n_events, k), np.inf)
        at = 0
        for e, size in zip(picked, sizes):
            order = at + np.argsort(score[at:at + size], kind="stable")[:k]
            want_i[e, :order.size], want_s[e, :order.size] = order, score[order]
            at += size
        np.testing.assert_array_equal(idx, want_i)
        np.testing.assert_array_equal(sc, want_s)
    c.close()
