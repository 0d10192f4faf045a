"""The plan at sizes around its sort tiles (4096 rows), with runs that span many tiles, 32- and 64-bit
binning keys, dropped rows, and rows equidistant from planes; every integer equal to the oracle's."""
import numpy as np
import pytest

import synth
from oracle import plan as oplan

torch = pytest.importorskip("torch")
pg = pytest.importorskip("paper_2206_15117_amd.polgrid")

pytestmark = pytest.mark.gpu


def geometry(n=64, os=4, planes=5, support=6, tile=5, w_max=10.0):
    return synth.Geometry(n=n, cell=0.064 / n, os=os, w_planes=synth.linear_w_planes(planes, w_max),
                          support=np.full(planes, support, np.int32), tile=np.full(planes, tile, np.int32), mk=16)


def check(geom, uvw, chunk):
    k = pg.kernels_alloc(geom, 1)
    p = pg.plan(k, torch.from_numpy(uvw).cuda(), max_chunk=chunk)
    # the library drops rows with a coordinate that is not finite; the oracle drops what is off the grid
    want = oplan.plan(geom, np.where(np.isfinite(uvw).all(axis=1)[:, None], uvw, 1e9), chunk)
    perm, fine, items = (a.cpu().numpy() for a in p.arrays())
    assert (p.n_kept, p.n_dropped, p.n_items) == (want["n_kept"], want["n_dropped"], len(want["items"]))
    assert np.array_equal(perm, want["perm"])
    kept = want["perm"][:p.n_kept]
    assert np.array_equal(fine, np.stack([want["loc"]["fine_x"][kept], want["loc"]["fine_y"][kept]], axis=1))
    t = geom.tile[want["items"][:, 0]]
    got = np.stack([items[:, 0], items[:, 1] // t, items[:, 2] // t, items[:, 3], items[:, 4]], axis=1)
    assert np.array_equal(got, want["items"]) and not items[:, 5:].any()


def rows(geom, count, spread, seed):
    rng = np.random.default_rng(seed)
    half = geom.n / 2 / (geom.n * geom.cell)
    return np.stack([rng.uniform(-spread, spread, count) * half, rng.uniform(-spread, spread, count) * half,
                     rng.uniform(-12.0, 12.0, count)], axis=1)


@pytest.mark.parametrize("count", [1, 2, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 8192, 12289, 70001, (1 << 20) - 1, (1 << 20) + 16385])
def test_counts_around_the_tiles(count):
    g = geometry()
    check(g, rows(g, count, 1.1, count), 100)


@pytest.mark.parametrize("chunk", [1, 7, 1024, 1 << 30])
def test_runs_over_many_tiles(chunk):
    """290 000 rows in two bins: runs of up to 70 tiles, one starting inside a tile."""
    g = geometry(planes=2, tile=50, os=2)
    uvw = rows(g, 290000 if chunk > 1 else 20000, 0.2, 3)
    uvw[:, 2] = np.where(np.arange(len(uvw)) % 29 == 0, -10.0, 10.0)
    check(g, uvw, chunk)


@pytest.mark.parametrize("planes,tile,n,os", [(3, 1, 64, 2), (40, 1, 4096, 16), (1000, 1, 2048, 8)])
def test_narrow_and_wide_keys(planes, tile, n, os):
    g = geometry(n=n, os=os, planes=planes, tile=tile, support=2)
    check(g, rows(g, 9000, 1.02, planes), 3)


def test_nothing_kept_and_non_finite_rows():
    g = geometry()
    uvw = rows(g, 5000, 0.9, 1)
    uvw[::3, 0] = np.nan
    uvw[1::3, 1] = 1e30
    uvw[2::7, 2] = np.inf
    check(g, uvw, 50)
    check(g, np.full((4100, 3), 1e9), 50)


def test_rows_between_planes_and_planes_closer_than_rounding():
    """Equal rounded distances go to the lowest plane, also among planes closer than the rounding of w."""
    g = geometry(planes=9, w_max=8.0)
    w = np.concatenate([g.w_planes, (g.w_planes[1:] + g.w_planes[:-1]) / 2, [-100.0, 100.0, 0.0]])
    uvw = np.zeros((len(w), 3))
    uvw[:, 2] = w
    check(g, uvw, 4)
    base = 1e15
    g2 = synth.Geometry(n=64, cell=1e-3, os=4, w_planes=np.array([-3.0, 1.0, 1.25, 1.5, 2.0, 2.125, 3.0]),
                        support=np.full(7, 6, np.int32), tile=np.full(7, 5, np.int32), mk=16)
    uvw = np.zeros((6, 3))
    uvw[:, 2] = [base, -base, base * 16, 1.4, 1.375, -1.0]
    check(g2, uvw, 4)
