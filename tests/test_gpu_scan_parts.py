"""The allocation-free scan of a set of windows whose chunks outnumber the argmin partials
that its work array holds: it runs in several launches, which must walk the windows alike,
so that every seed is scored once and the events' best is the best over all launches.

The partials take half of the 256 MiB array that the windows and one workgroup's minima
leave, 16 bytes each: 8 386 656 chunks of 64 seeds for 20 hits and 768 seeds a workgroup.
Two short steps per seed keep such a scan to a fraction of a second; the last launch is the
remainder. Scores and counts equal those of one launch (rkn_scan_windows) exactly: the same
chunks run the same steps, lists and distances.
"""
import numpy as np
import pytest

from paper_1908_01949_amd import synth

pytestmark = pytest.mark.gpu

N_HITS = 20
PARTS = ((256 << 20) - 4 * 256 - N_HITS * 768 * 4) // 2 // 16


@pytest.fixture(scope="module")
def rk():
    from paper_1908_01949_amd import rknscan
    rknscan.load_library()
    return rknscan


@pytest.fixture(scope="module")
def setup(rk, geo, sfield):
    evs = [synth.event_fixed_total(geo, sfield, k, n_total=N_HITS) for k in range(2)]
    c = rk.Context(0)
    c.upload_geometry(geo); c.upload_field(sfield); c.upload_hits(*synth.pack_events(evs))
    yield c, evs
    c.close()


@pytest.mark.parametrize("events,beyond", [(1, 96), (1, 1696), (2, 1696)])
def test_launches_of_one_scan_agree(rk, setup, events, beyond):
    """One window whose last launch has fewer chunks than the chip has waves (96: one per
    CU; 1696: one per wave), and a small window of one event before the long one."""
    import torch
    c, evs = setup
    m = -(-(PARTS + beyond) // 64)          # 8^4 m seeds: 64 m chunks
    hw = [0.05, 20.0, 3.0, 3.0, 30.0]
    rows = [(events - 1, 0, evs[events - 1].truth_seeds[0], hw, [8, 8, 8, 8, m])]
    if events == 2:
        rows.insert(0, (0, 0, evs[0].truth_seeds[0], hw, [3, 3, 3, 3, 2]))
    w = synth.make_windows(rows)
    assert rk.rkn_scan_shape(c.ctx, rk.make_scan_params(n_steps=2)) == (6, 768)
    assert PARTS < 64 * m < PARTS + 3072
    n = int(sum(np.prod(x["count"].astype(np.int64)) for x in w))
    p = rk.make_scan_params(n_steps=2, precision=32, ptr_flags=rk.RKN_PTR_DEVICE)
    got = []
    for scan in (rk.rkn_scan_windows, rk.rkn_scan_windows_noalloc):
        out = (torch.full((n,), -1.0, dtype=torch.float64, device="cuda"),
               torch.full((n,), -1, dtype=torch.int32, device="cuda"),
               torch.full((2,), -7, dtype=torch.int64, device="cuda"),
               torch.full((2,), -1.0, dtype=torch.float64, device="cuda"))
        torch.cuda.synchronize()
        scan(c.ctx, p, w, *out)
        rk.rkn_synchronize(c.ctx)
        got.append(out)
    one, parts = got
    assert int((parts[1] < 0).sum()) == 0, "seeds that no launch scored"
    for a, b in zip(one, parts):
        assert torch.equal(a, b)
    first = n - 4096 * m                     # the long window's first seed
    best = int(torch.argmin(one[0][first:])) + first
    assert int(parts[2][events - 1]) == best and float(parts[3][events - 1]) == float(one[0][best])
