"""Reprojection and weight normalisation at the edges of their tiles: images smaller and larger than a 64 x 16
tile by one pixel, every number of planes, accumulation over pixels that receive nothing (outside the
field, under zero weights, under a NaN sample), and planes that do not start on 16 bytes.

Tolerance: float64 until one rounding of the sample (2^-24 of it) and, accumulated, one of the sum (2^-24 of
it); source coordinates agree to 1e-12 pixel, on samples of a few units."""
import math

import numpy as np
import pytest

from oracle import mosaic as omos
from paper_2206_15117_amd import mosaic as mos

torch = pytest.importorskip("torch")
pg = pytest.importorskip("paper_2206_15117_amd.polgrid")

pytestmark = pytest.mark.gpu
DEG = math.pi / 180.0
U = 2.0 ** -24 * 1.001


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("n_src,n_dst,npol", [(2, 2, 1), (15, 17, 3), (64, 63, 2), (65, 129, 4), (100, 66, 1)])
@pytest.mark.parametrize("weighted", [False, True])
def test_reproject_sizes(n_src, n_dst, npol, weighted):
    rng = np.random.default_rng(n_src * 1000 + n_dst + npol)
    sf = mos.SkyFrame(n_src, 1.3 * DEG / n_src, 1.0, 0.3)
    df = mos.SkyFrame(n_dst, 1.5 * DEG / n_dst, 1.0 + 0.2 * DEG, 0.3 - 0.1 * DEG)
    src = rng.standard_normal((npol, n_src, n_src)).astype(np.float32)
    wsrc = rng.uniform(0.2, 1.0, (n_src, n_src)).astype(np.float32)
    wsrc[: n_src // 2, : n_src // 3] = 0.0
    w64 = wsrc.astype(np.float64) if weighted else None
    want, want_w = omos.reproject(src.astype(np.float64), tuple(sf), tuple(df), w64)
    out = torch.full((npol, n_dst, n_dst), 7.0, device="cuda")
    ow = torch.full((n_dst, n_dst), 7.0, device="cuda")
    dw = dev(wsrc) if weighted else None
    pg.reproject(dev(src), sf, out, df, src_weight=dw, dst_weight=ow)
    assert (np.abs(out.cpu().numpy() - want) <= U * np.abs(want) + 1e-11).all()
    assert (np.abs(ow.cpu().numpy() - want_w) <= U * np.abs(want_w) + 1e-11).all()
    base = rng.standard_normal(out.shape).astype(np.float32)
    bw = rng.uniform(0, 1, ow.shape).astype(np.float32)
    out, ow = dev(base), dev(bw)
    pg.reproject(dev(src), sf, out, df, src_weight=dw, dst_weight=ow, accumulate=True)
    for got, b, add in ((out, base, want_w * want), (ow, bw, want_w)):
        sum64 = b.astype(np.float64) + add
        assert (np.abs(got.cpu().numpy() - sum64) <= U * (np.abs(add) + np.abs(sum64)) + 1e-11).all()
    # a NaN sample reaches the pixels it is a neighbour of, whatever its weight
    src[:, 0, 0] = np.nan
    nan_want = np.isnan(omos.reproject(src.astype(np.float64), tuple(sf), tuple(df), w64)[0])
    out = dev(base)
    pg.reproject(dev(src), sf, out, df, src_weight=dw, accumulate=True)
    assert np.array_equal(np.isnan(out.cpu().numpy()), nan_want)


@pytest.mark.parametrize("n,npol,shift", [(1, 1, 0), (7, 4, 0), (16, 3, 0), (16, 4, 1), (66, 2, 2)])
def test_weight_normalise_sizes(n, npol, shift):
    rng = np.random.default_rng(n + npol)
    img = rng.standard_normal((npol, n, n)).astype(np.float32)
    w = rng.uniform(0, 2, (n, n)).astype(np.float32)
    w[: n // 2] = 0.0
    img[:, 0, 0] = np.nan  # below the weight: cleared, not divided
    w[0, 0] = 0.1
    buf = torch.zeros(npol * n * n + shift, device="cuda")
    view = buf[shift:].view(npol, n, n)
    view.copy_(dev(img))
    got = pg.weight_normalise(view, dev(w), 0.25).cpu().numpy()
    want = np.where(w >= 0.25, img.astype(np.float64) / np.where(w > 0, w, 1), 0)
    assert (np.abs(got - want) <= U * np.abs(want)).all()
