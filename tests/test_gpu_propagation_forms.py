"""The refinement's forward pass and the scan in their three forms: few chunks in the field
map (seeds on four lanes of a wave), more (one lane, producer and consumer waves) and many
(waves that do both): the same results bit for bit.

The same seeds in the same chunks of 64 are passed once alone and once followed by enough
other chunks of their event. The lists, and with them every rounding, are then the same, so
residuals, Phi, argmin chords (through the gradient) and checkpoints (through the gradient
and J^T J, recomputed from them) are compared exactly, and so are the scan's scores.
"""
import numpy as np
import pytest

from paper_1908_01949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rk():
    from paper_1908_01949_amd import rknscan
    rknscan.load_library()
    return rknscan


@pytest.fixture(scope="module")
def setup(rk, geo, ufield, sfield):
    ev = synth.event_multi_turn(geo, ufield, 3)
    c = rk.Context(0)
    c.upload_geometry(geo); c.upload_field(sfield); c.upload_hits(*synth.pack_events([ev]))
    yield c, ev
    c.close()


def _seeds(ev, n, scale):
    return np.asarray(ev.truth_seeds[0]) + np.array(scale) * np.random.default_rng(7).uniform(-1, 1, (n, 5))


@pytest.mark.parametrize("turn_stop", [0, 1])
def test_refinement(rk, setup, turn_stop):
    """128 seeds on four lanes; among 19 264 (301 chunks, two pairs a CU) and 64 064 (1001
    chunks) on one."""
    c, ev = setup
    s = _seeds(ev, 64064, (0.003, 10.0, 0.6, 0.6, 0.6))
    p = rk.make_scan_params(n_steps=1003, precision=32, turn_stop=turn_stop)

    def run(n):
        rk.rkn_refine_setup(c.ctx, p, np.zeros(n, np.int32), s[:n], 64)
        r = np.zeros((n, c.max_hits), np.float32); phi = np.zeros(n)
        g = np.zeros((n, 5)); S = np.zeros((n, 5, 5))
        rk.rkn_residuals_fwd(c.ctx, None, r, phi)
        rk.rkn_adjoint_bwd(c.ctx, None, g, S)
        return [x[:128].copy() for x in (r, phi, g, S)]
    quad = run(128)
    assert np.count_nonzero(np.isfinite(quad[0])) > 128 and np.abs(quad[2]).max() > 0
    for n in (19264, 64064):
        for a, b in zip(quad, run(n)):
            assert np.array_equal(a, b, equal_nan=True), n


@pytest.mark.parametrize("block_steps", [4, 6, 8])
@pytest.mark.parametrize("turn_stop", [0, 1])
def test_scan(rk, setup, block_steps, turn_stop):
    """Scores of tracks that stay within the wires' z range (so that no launch skips a
    block), among 12 800 seeds (four lanes), 19 264 and 256 000 (one)."""
    c, ev = setup
    s = _seeds(ev, 256000, (0.05, 60.0, 6.0, 6.0, 1.0))
    p = rk.make_scan_params(n_steps=403, precision=32, turn_stop=turn_stop, block_steps=block_steps)

    def run(n):
        out = (np.zeros(n), np.zeros(n, np.int32), np.zeros(1, np.int64), np.zeros(1))
        rk.rkn_scan_seeds(c.ctx, p, np.zeros(n, np.int32), s[:n], *out)
        return out[0][:12800], out[1][:12800]
    quad = run(12800)
    for n in (19264, 256000):
        for a, b in zip(quad, run(n)):
            assert np.array_equal(a, b), n
