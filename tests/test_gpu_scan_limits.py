"""Which scans the LDS admits, and in which shape: the limits do not depend on how many
seeds a call has, and the bookkeeping of a workgroup's chunks does not narrow them.

LDS of a workgroup of W waves with B-step blocks (FP32, field map nr x nz, L layers, h hits
in the largest event), bytes: 8 (nr + 1)(nz + 1) and 32 h, each rounded up to 64; 2048;
512 L; W (B + 1) 768; 704 W; 4 (2 L + 1); 4 W ceil(h / 32). A shape is taken when 256 more
fit the 160 KiB (272 more for 16 waves).
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


def _hits(geo, h):
    rng = np.random.default_rng(h)
    return (np.array([0, h], np.int32), np.sort(rng.choice(geo.mx.size, h, replace=False)).astype(np.int32),
            rng.uniform(0, 8, h).astype(np.float32))


@pytest.mark.parametrize("block_steps,hits,lanes", [(6, 314, 768), (6, 315, 512), (4, 316, 1024), (4, 317, 512)])
def test_widest_shape_up_to_its_limit(rk, geo, sfield, block_steps, hits, lanes):
    """The 18-layer chamber: 12 waves up to 314 hits, 16 waves up to 316."""
    c = rk.Context(0)
    c.upload_geometry(geo); c.upload_field(sfield); c.upload_hits(*_hits(geo, hits))
    assert rk.rkn_scan_shape(c.ctx, rk.make_scan_params(precision=32, block_steps=block_steps)) == (block_steps, lanes)
    c.close()


@pytest.mark.parametrize("precision,nr,scans,refines", [(32, 80, True, True), (32, 84, True, False),
                                                        (32, 92, True, False), (32, 96, False, False),
                                                        (64, 104, True, None), (64, 108, False, None)])
def test_maps_past_the_limit_are_refused_for_any_number_of_seeds(rk, geo, precision, nr, scans, refines):
    """Maps of nr x 129 nodes, 18 layers, 100 hits: a map that leaves the scan's workgroup
    (6-step blocks of 8 waves, FP64: 4-step blocks of 4) or the refinement's (8-step blocks
    of 8 waves) no room is refused, few seeds or many."""
    field = synth.constant_grid_field(1.0, nr=nr, nz=129)
    c = rk.Context(0)
    c.upload_geometry(geo); c.upload_field(field); c.upload_hits(*_hits(geo, 100))
    p = rk.make_scan_params(n_steps=20, precision=precision)
    rng = np.random.default_rng(0)
    for n in (1, 100, 40000):
        s = np.array([0.3, 0.0, 60.0, 70.0, 5.0]) + rng.uniform(-1, 1, (n, 5))
        e = np.zeros(n, np.int32)
        out = (np.zeros(n), np.zeros(n, np.int32), np.zeros(1, np.int64), np.zeros(1))
        calls = [(scans, lambda: rk.rkn_scan_seeds(c.ctx, p, e, s, *out))]
        if precision == 32 and n <= 100:
            calls += [(refines, lambda: rk.rkn_classify_hits(c.ctx, p, e, s, c.max_hits)),
                      (refines, lambda: rk.rkn_refine_setup(c.ctx, p, e, s, 8))]
        for fits, call in calls:
            if fits:
                call()
            else:
                with pytest.raises(rk.RknError) as err:
                    call()
                assert err.value.status in (rk.RKN_E_UNSUPPORTED, rk.RKN_E_DEVICE)
    c.close()
