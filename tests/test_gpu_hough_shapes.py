"""Hough accumulator and windows over grid shapes: cell counts below, at and past a vote
workgroup's 256 and off a multiple of 8, one radius bin to the largest number, bins so
narrow (2^-8 mm) that the FP32 estimate of the bin decides nothing, and events of no hits
to the largest number. Whole numbers, so compared exactly with the oracle."""
import numpy as np
import pytest

from paper_1908_01949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hits(geo, ufield):
    evs = [synth.event_fixed_total(geo, ufield, s, n_total=150, noise_frac=0.2) for s in (1, 2)]
    off, wid, dr = synth.pack_events(evs)
    many = np.random.default_rng(0).permutation(geo.n_wires)[:512].astype(np.int32)   # the largest event
    # one hit; none; the two tracks; the largest
    return (np.concatenate([[0, 1], off + 1, off[-1:] + 513]).astype(np.int32),
            np.concatenate([many[:1], wid, many]), np.concatenate([dr[:1], dr, np.ones(512, np.float32)]))


@pytest.mark.parametrize("n_xy,n_r,xy_half,r_min,r_max", [
    (1, 1, 512.0, 160.0, 416.0), (2, 3, 512.0, 0.0, 768.0), (15, 64, 480.0, 160.0, 416.0), (16, 5, 512.0, 160.0, 480.0),
    (17, 63, 544.0, 100.0, 352.0), (33, 2, 528.0, 8.0, 600.0), (64, 64, 512.0, 300.0, 300.25),
    (255, 17, 510.0, 160.0, 432.0)])
def test_accumulator_and_windows_equal_the_oracle(geo, ufield, orc_u, hits, n_xy, n_r, xy_half, r_min, r_max):
    from paper_1908_01949_amd import rknscan as rk
    off, wid, dr = hits
    kw = dict(n_xy=n_xy, n_r=n_r, xy_half=xy_half, r_min=r_min, r_max=r_max, min_votes=3, max_cand=7)
    hp, ohp = rk.make_hough_params(**kw), orc_u.hough_params(**kw)
    c = rk.Context(0)
    c.upload_geometry(geo); c.upload_field(ufield); c.upload_hits(off, wid, dr)
    for e in range(off.size - 1):
        g = rk.rkn_hough_accumulator(c.ctx, hp, e)
        np.testing.assert_array_equal(g, orc_u.hough_accumulate(ohp, wid[off[e]:off[e + 1]]))
    g = rk.rkn_hough_seed_windows(c.ctx, hp)
    o = orc_u.hough_seed_windows(ohp, off, wid)
    for name in ("event", "candidate", "count"):
        np.testing.assert_array_equal(g[name], o[name])
    np.testing.assert_allclose(g["center"], o["center"], rtol=0, atol=1e-11)
    c.close()
