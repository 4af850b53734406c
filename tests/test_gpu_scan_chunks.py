"""GPU scan at the edges of its work division: chunks of 64 seeds (one wave each) with and
without a remainder, launches of a few chunks (propagation and culling side by side) and
of many, the z range past which blocks are skipped, and the refinement pass's point
columns (16, 48 or 64 seeds per event).

Tolerances: scores and n_in against the FP64 oracle by the rules of parity_util; the two
forms of the kernel against each other 1e-6 relative, since they run the same FP32 steps
and distances and may only differ by the rounding order of one product sum per distance
(1 ulp of a closest-approach parameter, second order in the distance); residuals of the
same seed in differently filled chunks 1e-4 mm for the same reason.
"""
import numpy as np
import pytest

from paper_1908_01949_amd import synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rk():
    from paper_1908_01949_amd import rknscan
    rknscan.load_library()
    return rknscan


@pytest.fixture(scope="module")
def setups(rk, geo, ufield, sfield, orc_u, orc_s):
    out = {}
    for name, field, O in (("u", ufield, orc_u), ("s", sfield, orc_s)):
        evs = [synth.event_multi_turn(geo, ufield, k) for k in (3, 4)]
        off, wid, dr = synth.pack_events(evs)
        c = rk.Context(0)
        c.upload_geometry(geo); c.upload_field(field); c.upload_hits(off, wid, dr)
        out[name] = (c, O, evs, (off, wid, dr))
    yield out
    for c, *_ in out.values():
        c.close()


def _seeds(evs, n, rng, scale=(0.05, 60.0, 6.0, 6.0, 6.0)):
    e = np.sort(rng.integers(0, len(evs), n)).astype(np.int32)
    base = np.stack([evs[i].truth_seeds[0] for i in e])
    return e, base + np.array(scale) * rng.uniform(-1, 1, (n, 5))


def _scan(rk, c, p, e, s, n_events=2):
    out = (np.zeros(len(e)), np.zeros(len(e), np.int32), np.zeros(n_events, np.int64), np.zeros(n_events))
    rk.rkn_scan_seeds(c.ctx, p, e, s, *out)
    return out


@pytest.mark.parametrize("turn_stop", [0, 1])
@pytest.mark.parametrize("fieldname,precision", [("u", 32), ("u", 64), ("s", 32), ("s", 64)])
@pytest.mark.parametrize("n", [1, 63, 65, 130])
def test_few_chunks_match_oracle(rk, setups, fieldname, precision, n, turn_stop):
    """1003 steps: the last block of 4, 6 or 8 steps is short."""
    c, O, evs, hits = setups[fieldname]
    e, s = _seeds(evs, n, np.random.default_rng(n))
    p = rk.make_scan_params(n_steps=1003, precision=precision, turn_stop=turn_stop)
    score, nin, bi, bs = _scan(rk, c, p, e, s)
    osc, onin, obi, _ = O.scan_seeds(O.params(n_steps=1003, turn_stop=turn_stop), *hits, e, s, mode=1)
    pu.check_scores(score, osc)
    pu.check_nin(nin, onin)
    for k in range(2):
        at = np.nonzero(e == k)[0]
        if at.size == 0:
            assert bi[k] == -1 and np.isinf(bs[k])
        else:
            assert bs[k] == score[at].min() and score[bi[k]] == bs[k] and e[bi[k]] == k


@pytest.mark.parametrize("fieldname", ["u", "s"])
def test_many_chunks_equal_few(rk, setups, fieldname):
    """A window of more chunks than fit the chip at once, in counts that leave remainders,
    against its own seeds scanned a few at a time."""
    c, _, evs, _ = setups[fieldname]
    count = [9, 11, 9, 10, 11]
    w = synth.make_windows([(k, 0, evs[k].truth_seeds[0], [0.1, 80, 8, 8, 30], count) for k in range(2)])
    size = int(np.prod(count))
    p = rk.make_scan_params(n_steps=400, precision=32)
    score = np.zeros(2 * size); nin = np.zeros(2 * size, np.int32)
    bi = np.zeros(2, np.int64); bs = np.zeros(2)
    rk.rkn_scan_windows(c.ctx, p, w, score, nin, bi, bs)
    rng = np.random.default_rng(5)
    g = np.sort(rng.choice(2 * size, 400, replace=False))
    grid = [np.stack(np.meshgrid(*[np.linspace(a - h, a + h, m) for a, h, m in
                                   zip(w[k]["center"], w[k]["half_width"], count)], indexing="ij"), -1).reshape(-1, 5)
            for k in range(2)]
    few, few_n, _, _ = _scan(rk, c, p, (g // size).astype(np.int32), np.concatenate(grid)[g])
    assert np.all(np.abs(few - score[g]) <= 1e-6 * score[g] + 1e-6)
    assert np.abs(few_n - nin[g]).max() <= 1
    for k in range(2):
        part = score[k * size:(k + 1) * size]
        assert bi[k] == k * size + int(np.argmin(part)) and bs[k] == part.min()


@pytest.mark.parametrize("n", [40, 70000])
@pytest.mark.parametrize("fieldname", ["u", "s"])
def test_tracks_leaving_in_z(rk, setups, fieldname, n):
    """Steep tracks from seeds near and past the chamber's ends: blocks out of the wires'
    reach along z are skipped, tracks that enter it late are not."""
    c, O, evs, hits = setups[fieldname]
    rng = np.random.default_rng(n)
    e, s = _seeds(evs, n, rng)
    s[:, 1] = rng.uniform(-1100, 1100, n)
    s[:, 4] = rng.uniform(-80, 80, n)
    p = rk.make_scan_params(n_steps=2500, precision=32)
    score, nin, _, _ = _scan(rk, c, p, e, s)
    at = np.sort(rng.choice(n, 40, replace=False))
    osc, onin, _, _ = O.scan_seeds(O.params(n_steps=2500), *hits, e[at], s[at], mode=1)
    pu.check_scores(score[at], osc)
    pu.check_nin(nin[at], onin)


@pytest.mark.parametrize("fieldname", ["u", "s"])
@pytest.mark.parametrize("n", [16, 17, 48, 49, 65])
def test_refinement_columns(rk, setups, fieldname, n):
    """The residuals of an event's seeds do not depend on how many of them there are."""
    c, _, evs, _ = setups[fieldname]
    _, s = _seeds(evs[:1], n, np.random.default_rng(n), scale=(0.003, 10.0, 0.6, 0.6, 0.6))
    p = rk.make_scan_params(n_steps=2003, precision=32)

    def residuals(rows):
        rk.rkn_refine_setup(c.ctx, p, np.zeros(len(rows), np.int32), s[rows], 64)
        r = np.zeros((len(rows), c.max_hits), np.float32); phi = np.zeros(len(rows))
        rk.rkn_residuals_fwd(c.ctx, None, r, phi)
        return r, phi
    r, phi = residuals(list(range(n)))
    for k in (0, n // 2, n - 1):
        r1, phi1 = residuals([k])
        assert np.array_equal(np.isnan(r[k]), np.isnan(r1[0]))
        assert np.nanmax(np.abs(r[k] - r1[0])) <= 1e-4
        assert abs(phi[k] - phi1[0]) <= 1e-3 * phi1[0] + 1e-6
