"""Edges of the exchange's work split, beside the shapes of the exchange tests.

Sums: few large boxes, where a workgroup adds up thousands of partial sums: whole
spheres in two intervals of unequal length (one box has fewer levels than there
are sums over levels), the sums of a box below and above the count from which
16 waves share them.

Orders: pieces stay in rows below 56 columns and go by the set of boxes that
share a cell from there on: 55 and 56 columns, bricks on both sides of it, bands
around the circle, and rows most of which are shared."""
import pytest

import test_gpu_exchange as exchange

pytestmark = pytest.mark.gpu

SPHERES = dict(nsteps=9, bands=1, pieces=1, ntime=2, overlap_cells=0, overlap_steps=2, obs_frac=0.01)
ORDERS = {
    "columns_55": dict(nlat=20, nlon=102),
    "columns_56": dict(nlat=20, nlon=104),
    "bricks": dict(nlat=40, nlon=270, brick=(2, 5, 12, 90), overlap_cells=3),
    "bands": dict(nlat=24, nlon=64, bands=3, pieces=1),
    "mostly_shared": dict(nlat=16, nlon=220, bands=2, pieces=4, overlap_cells=6),
}


@pytest.mark.parametrize("nlat, nlon, sums", [(64, 128, 1024), (96, 192, 2304)])
def test_sums_of_large_boxes(nlat, nlon, sums, monkeypatch):
    assert 4 * 8 * (nlat * nlon // 256) == sums
    monkeypatch.setitem(exchange.CASES, "spheres", dict(SPHERES, nlat=nlat, nlon=nlon))
    exchange.test_exchange_edges("spheres")


@pytest.mark.parametrize("which", list(ORDERS))
def test_orders(which, monkeypatch):
    monkeypatch.setitem(exchange.CASES, which, ORDERS[which])
    exchange.test_exchange_edges(which)
