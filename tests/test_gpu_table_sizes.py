"""Kernel tables against the float64 oracle at the sizes where the generator's tiling can go wrong: lattices
and table sides that are not multiples of its 32-wide tiles and 16-deep slices (and smaller than one),
sets of more planes than one round of launches takes, one and two Jones fields, both kinds and storages.

Tolerance: the transform is float64, so an entry is off by the rounding to storage: 2^-24 of a float32
component, 2^-11 of a float16 component (2^-25 below its normal range), and 1e-11 of the largest entry for
the two float64 transforms' own rounding."""
import numpy as np
import pytest

import synth
from oracle import kernels, mueller
from test_gpu_parity import gpu_layout

torch = pytest.importorskip("torch")
pg = pytest.importorskip("paper_2206_15117_amd.polgrid")

pytestmark = pytest.mark.gpu

CASES = [
    # mk, os, support per plane, npol, fields, direction, storage
    (2, 2, [1], 1, 0, "grid", 0),
    (2, 2, [1, 2], 4, 1, "grid", 0),
    (18, 2, [8, 3, 5], 4, 2, "grid", 0),
    (34, 4, [8, 9], 4, 1, "degrid", 1),
    (50, 6, [5, 6, 7], 4, 2, "degrid", 0),
    (64, 8, [6, 7, 8, 4, 5, 6, 7, 8, 4, 6, 5], 1, 0, "grid", 1),
    (30, 16, [2, 3], 4, 0, "grid", 0),
    (130, 4, [17, 11, 24], 4, 1, "grid", 1),
]


@pytest.mark.parametrize("mk,os_,support,npol,fields,direction,storage", CASES)
@pytest.mark.parametrize("convention", ["iau", "paper"])
def test_tables_match_the_oracle(mk, os_, support, npol, fields, direction, storage, convention):
    pg.use_torch_allocator(True)
    rng = np.random.default_rng(mk * os_ + npol)
    n = 128
    planes = len(support)
    g = synth.Geometry(n, 0.06 / n, os_, 40.0 * (np.arange(planes) - 0.5 * (planes - 1)), np.array(support),
                       tile=np.full(planes, 16), mk=mk)
    jones = []
    for _ in range(fields):
        j = 0.1 * (rng.standard_normal((2, 2, mk, mk)) + 1j * rng.standard_normal((2, 2, mk, mk)))
        j[0, 0] += rng.uniform(0.1, 1.0, (mk, mk))
        j[1, 1] += rng.uniform(0.1, 1.0, (mk, mk))
        jones.append(j)
    ja = jones[0] if fields else None
    jb = jones[1] if fields == 2 else None
    kind = pg.KIND_GRID if direction == "grid" else pg.KIND_DEGRID
    if npol == 1 or fields == 0:
        phi = mueller.phi_identity(npol, mk, mk, direction, 0.2, convention)
    elif direction == "grid":
        phi = mueller.phi_grid(ja, 0.2, convention, jones_b=jb)
    else:
        phi = mueller.phi_degrid(ja, convention, jones_b=jb)
    want = gpu_layout(kernels.make_tables(g, phi), entries=4 if storage else 2)
    conv = pg.STOKES_IAU if convention == "iau" else pg.STOKES_PAPER
    k = pg.make_kernels(g, npol, kind, jones=ja, jones_b=jb, eps_null=0.2, storage=storage, convention=conv)
    got = k.table().cpu().numpy()
    if got.dtype != np.complex64:
        got = got.astype(np.float64).reshape(-1, 2)
        got = got[:, 0] + 1j * got[:, 1]
    assert got.shape == want.shape
    unit, floor = (2.0 ** -11, 2.0 ** -25) if storage else (2.0 ** -24, 0.0)
    slack = floor + 1e-11 * np.abs(want).max()
    assert (np.abs(got.real - want.real) <= unit * np.abs(want.real) + slack).all()
    assert (np.abs(got.imag - want.imag) <= unit * np.abs(want.imag) + slack).all()


@pytest.mark.parametrize("ja,jb,eps,refused", [
    ([1, 1, 1, 1], [1, 1, 1, 1], 0.0, True),      # rank one: a pivot of exactly zero
    ([1, 1, 1, 1], [1, 1, 1, 1], 0.2, False),     # regularised
    ([0, 0, 0, 0], [0, 0, 0, 0], 0.0, False),     # a null diagonal is replaced, not refused
    ([0, 0, 0, 0.1], [-1, 1 + 1j, -1, 0.1], 0.0, False),  # rank one, but rounding leaves no zero
    ([1e-170, 1, 1, 0.5], [1, 0, 0, 1], 0.2, False),
    ([np.nan, 0, 0, 1], [1, 0, 0, 1], 0.2, False),
])
def test_singular_fields_are_refused_by_their_pivots(ja, jb, eps, refused):
    pg.use_torch_allocator(True)
    mk = 4
    g = synth.Geometry(64, 1e-3, 2, np.zeros(1), np.array([3]), tile=np.array([8]), mk=mk)
    fields = [np.ascontiguousarray(np.broadcast_to(np.array(j, dtype=complex).reshape(2, 2, 1, 1), (2, 2, mk, mk))) for j in (ja, jb)]
    if refused:
        with pytest.raises(pg.PolgridError):
            pg.make_kernels(g, 4, pg.KIND_GRID, jones=fields[0], jones_b=fields[1], eps_null=eps)
    else:
        pg.make_kernels(g, 4, pg.KIND_GRID, jones=fields[0], jones_b=fields[1], eps_null=eps)
