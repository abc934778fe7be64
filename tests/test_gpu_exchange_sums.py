"""The overlap constant of J on few large boxes, where a workgroup adds up
thousands of partial sums: whole spheres in two intervals of unequal length
(one box has fewer levels than there are sums over levels), with the sums of a
box below and above the count from which 16 waves share them."""
import pytest

import test_gpu_exchange as exchange

pytestmark = pytest.mark.gpu

SPHERES = dict(nsteps=9, bands=1, pieces=1, ntime=2, overlap_cells=0, overlap_steps=2, obs_frac=0.01)


@pytest.mark.parametrize("nlat, nlon, sums", [(64, 128, 1024), (96, 192, 2304)])
def test_sums_of_large_boxes(nlat, nlon, sums, monkeypatch):
    assert 4 * 8 * (nlat * nlon // 256) == sums
    monkeypatch.setitem(exchange.CASES, "spheres", dict(SPHERES, nlat=nlat, nlon=nlon))
    exchange.test_exchange_edges("spheres")
